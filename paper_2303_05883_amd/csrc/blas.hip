// Fused vector kernels and deterministic reductions of the BiCGStab solver.
//
// Every update kernel reads the solver's scalars (alpha, beta, omega) from
// device memory, so an iteration needs no host round trip and can be replayed
// from a captured graph; every kernel first checks the solve's "done" flag and
// returns at once when it is set. Reductions are FP64: each block writes its
// partial sums in a fixed slot, and a one-block finalize kernel, or on small
// lattices the next update kernel itself (Fold), adds them in a fixed order, so
// repeated FP64 runs are bitwise identical. They also compute the next scalars (the solver's global reductions, of up
// to three values at once, the pattern the paper credits for solver
// efficiency in Sec. 3).
#include "blascore.h"

namespace lq {

namespace {

constexpr int BS = 256;
constexpr int FBS = 1024;  // threads of the one-block finalize kernels

// done, in a launch that may set it itself (fold: before the barriers of its sums) or not
__device__ inline bool is_done(const Scal* s, bool fold) { return fold ? group_flag(&s->done) : s->done != 0; }

// p = r + beta (p - omega v); with f, after forming beta from the sums of <rhat, r>, <r, r>
template <int P>
__global__ void __launch_bounds__(BS) k_p_update(const void* r, void* p, const void* v, Scal* sc, Fold f, size_t vh) {
  if (is_done(sc, f.n != 0)) return;
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
  cx<double> beta = {sc->beta_r, sc->beta_i};
  if (f.n) {
    double s[3];
    sum_partials<3>(f.partials, f.n, s);
    const int end = beta_of(sc, s, beta);
    if (lead) {
      sc->next_r = s[0];
      sc->next_i = s[1];
      scal_count(sc, s[2], end);
    }
    if (end) return;
  }
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i < vh) p_update_site<P>(r, p, v, beta, {sc->omega_r, sc->omega_i}, i);
}

// s = r - alpha v; with f, after forming alpha from the sums of <rhat, v>
template <int P>
__global__ void __launch_bounds__(BS) k_s_update(const void* r, const void* v, void* s, Scal* sc, Fold f, size_t vh) {
  if (is_done(sc, f.n != 0)) return;
  cx<double> alpha = {sc->alpha_r, sc->alpha_i};
  if (f.n) {
    const cx<double> rho = {sc->next_r, sc->next_i};
    double d[2];
    sum_partials<2>(f.partials, f.n, d);
    const bool ok = alpha_of(rho, d, alpha);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sc->rho_r = rho.r;
      sc->rho_i = rho.i;
      if (ok) {
        sc->alpha_r = alpha.r;
        sc->alpha_i = alpha.i;
      } else {
        scal_stop(sc, true);
      }
    }
    if (!ok) return;
  }
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i < vh) s_update_site<P>(r, v, s, alpha, i);
}

// x += alpha p + omega s (x in precision PX); r = s - omega t; partials <rhat, r>, <r, r>;
// with f, after forming omega from the sums of <t, s>, <t, t>
template <int P, int PX>
__global__ void __launch_bounds__(BS) k_xr_update(void* x, const void* p, const void* s, const void* t, void* r,
                                                  const void* rhat, Scal* sc, Fold f, double* partials, size_t vh) {
  if (is_done(sc, f.n != 0)) return;
  cx<double> omega = {sc->omega_r, sc->omega_i};
  if (f.n) {
    double d[3];
    sum_partials<3>(f.partials, f.n, d);
    omega = omega_of(d);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sc->omega_r = omega.r;
      sc->omega_i = omega.i;
    }
  }
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  double red[3] = {0.0, 0.0, 0.0};
  if (i < vh) xr_update_site<P, PX>(x, p, s, t, r, rhat, {sc->alpha_r, sc->alpha_i}, omega, i, red);
  block_reduce<3>(red, partials + (size_t)blockIdx.x * 3);
}

// partials <a, b> (re, im) and <b, b>
template <int P>
__global__ void __launch_bounds__(BS) k_dot_norm(const void* a, const void* b, double* partials, size_t vh) {
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  double red[3] = {0.0, 0.0, 0.0};
  if (i < vh) dot_norm_site<P>(a, b, i, red);
  block_reduce<3>(red, partials + (size_t)blockIdx.x * 3);
}

// out = a - b (FP64), partial ||out||^2
__global__ void __launch_bounds__(BS) k_sub_norm(const void* a, const void* b, void* out, double* partials, size_t vh) {
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  double red[1] = {0.0};
  if (i < vh) {
    cx<double> av[12], bv[12];
    IO<0>::load_spinor(a, i, av);
    IO<0>::load_spinor(b, i, bv);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      av[k] = av[k] - bv[k];
      red[0] += av[k].r * av[k].r + av[k].i * av[k].i;
    }
    IO<0>::store_spinor(out, i, av);
  }
  block_reduce<1>(red, partials + blockIdx.x);
}

// dst (precision PD) = scale * src (FP64); scale read from device (1 / ||r||) or given
template <int PD>
__global__ void __launch_bounds__(BS) k_scale_down(const void* src, void* dst, const double* dscale, double hscale,
                                                   size_t vh) {
  using TD = typename IO<PD>::T;
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i >= vh) return;
  const double s = dscale ? *dscale : hscale;
  cx<double> a[12];
  cx<TD> d[12];
  IO<0>::load_spinor(src, i, a);
#pragma unroll
  for (int k = 0; k < 12; ++k) d[k] = {(TD)(s * a[k].r), (TD)(s * a[k].i)};
  IO<PD>::store_spinor(dst, i, d);
}

// x64 += scale * e (e in precision PS)
template <int PS>
__global__ void __launch_bounds__(BS) k_accum_up(void* x, const void* e, const double* dscale, size_t vh) {
  using TS = typename IO<PS>::T;
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i >= vh) return;
  const double s = *dscale;
  cx<double> a[12];
  cx<TS> b[12];
  IO<0>::load_spinor(x, i, a);
  IO<PS>::load_spinor(e, i, b);
#pragma unroll
  for (int k = 0; k < 12; ++k) a[k] = a[k] + s * cx<double>{(double)b[k].r, (double)b[k].i};
  IO<0>::store_spinor(x, i, a);
}

template <int P>
__global__ void __launch_bounds__(BS) k_copy(const void* src, void* dst, size_t vh) {
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i < vh) copy_site<P>(src, dst, i);
}

template <int P>
__global__ void __launch_bounds__(BS) k_zero(void* dst, size_t vh) {
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i < vh) zero_site<P>(dst, i);
}

// p *= f, v *= f (a reliable update changes the residual's normalisation)
template <int P>
__global__ void __launch_bounds__(BS) k_scale2(void* p, void* v, double f, size_t vh) {
  using T = typename IO<P>::T;
  const size_t i = (size_t)blockIdx.x * BS + threadIdx.x;
  if (i >= vh) return;
  const T s = (T)f;
  cx<T> a[12];
  IO<P>::load_spinor(p, i, a);
#pragma unroll
  for (int k = 0; k < 12; ++k) a[k] = s * a[k];
  IO<P>::store_spinor(p, i, a);
  IO<P>::load_spinor(v, i, a);
#pragma unroll
  for (int k = 0; k < 12; ++k) a[k] = s * a[k];
  IO<P>::store_spinor(v, i, a);
}

__global__ void __launch_bounds__(FBS) k_fin_reliable(Scal* sc, const double* partials, int n, double target2) {
  double v[3];
  sum_partials<3>(partials, n, v);
  if (threadIdx.x == 0) scal_reliable(sc, v, target2);
}

// alpha = rho / <rhat, v>
__global__ void __launch_bounds__(FBS) k_fin_alpha(Scal* sc, const double* partials, int n) {
  if (sc->done) return;
  double v[2];
  sum_partials<2>(partials, n, v);
  if (threadIdx.x == 0) scal_alpha(sc, v);
}

// omega = <t, s> / <t, t>
__global__ void __launch_bounds__(FBS) k_fin_omega(Scal* sc, const double* partials, int n) {
  if (sc->done) return;
  double v[3];
  sum_partials<3>(partials, n, v);
  if (threadIdx.x == 0) scal_omega(sc, v);
}

// rho_new = <rhat, r>, rr = <r, r>; beta = (rho_new / rho)(alpha / omega); convergence test
__global__ void __launch_bounds__(FBS) k_fin_rho(Scal* sc, const double* partials, int n) {
  if (sc->done) return;
  double v[3];
  sum_partials<3>(partials, n, v);
  if (threadIdx.x == 0) scal_rho(sc, v);
}

// Start of a (re)start: rho = <rhat, r>, rr = <r, r>, alpha = omega = 1.
__global__ void __launch_bounds__(FBS) k_fin_init(Scal* sc, const double* partials, int n, double target2,
                                                  int max_iters) {
  double v[3];
  sum_partials<3>(partials, n, v);
  if (threadIdx.x == 0) scal_init(sc, v, target2, max_iters);
}

// out[0] = sum of n partials (width 1 or 3, component `comp`); out[1] = 1/sqrt(out[0]) (0 if out[0] == 0)
__global__ void __launch_bounds__(FBS) k_fin_norm(double* out, const double* partials, int n, int width, int comp) {
  double v = 0.0;
  for (int j = threadIdx.x; j < n; j += blockDim.x) v += partials[(size_t)j * width + comp];
  double tmp[1] = {v};
  __shared__ double res[1];
  block_reduce<1>(tmp, res);
  __syncthreads();
  if (threadIdx.x == 0) {
    out[0] = res[0];
    out[1] = res[0] > 0.0 ? 1.0 / sqrt(res[0]) : 0.0;
    out[2] = sqrt(res[0]);
  }
}

inline int nblk(size_t vh) { return (int)((vh + BS - 1) / BS); }

}  // namespace

int blas_blocks(size_t vh) { return nblk(vh); }

#define LQ_PREC_SWITCH(prec, CALL)                             \
  switch (prec) {                                              \
    case 0: { constexpr int P = 0; CALL; } break;              \
    case 1: { constexpr int P = 1; CALL; } break;              \
    case 2: { constexpr int P = 2; CALL; } break;              \
    default: return set_error(LQCD_EINVAL, "bad precision");   \
  }

int blas_p_update(lqcd_ctx* c, int prec, const void* r, void* p, const void* v, Scal* sc, Fold f) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_p_update<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, r, p, v, sc, f, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_s_update(lqcd_ctx* c, int prec, const void* r, const void* v, void* s, Scal* sc, Fold f) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_s_update<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, r, v, s, sc, f, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_xr_update(lqcd_ctx* c, int prec, int xprec, void* x, const void* p, const void* s, const void* t, void* r,
                   const void* rhat, Scal* sc, double* partials, Fold f) {
  const size_t vh = c->g.vh;
  const dim3 g(nblk(vh)), b(BS);
  if (prec == 0 && xprec == 0)
    hipLaunchKernelGGL((k_xr_update<0, 0>), g, b, 0, c->stream, x, p, s, t, r, rhat, sc, f, partials, vh);
  else if (prec == 1 && xprec == 1)
    hipLaunchKernelGGL((k_xr_update<1, 1>), g, b, 0, c->stream, x, p, s, t, r, rhat, sc, f, partials, vh);
  else if (prec == 2 && xprec == 1)
    hipLaunchKernelGGL((k_xr_update<2, 1>), g, b, 0, c->stream, x, p, s, t, r, rhat, sc, f, partials, vh);
  else if (prec == 2 && xprec == 2)
    hipLaunchKernelGGL((k_xr_update<2, 2>), g, b, 0, c->stream, x, p, s, t, r, rhat, sc, f, partials, vh);
  else
    return set_error(LQCD_EINVAL, "unsupported precision pair for x/r update");
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_dot_norm(lqcd_ctx* c, int prec, const void* a, const void* b, double* partials) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_dot_norm<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, a, b, partials, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_sub_norm(lqcd_ctx* c, const void* a, const void* b, void* out, double* partials) {
  const size_t vh = c->g.vh;
  hipLaunchKernelGGL(k_sub_norm, dim3(nblk(vh)), dim3(BS), 0, c->stream, a, b, out, partials, vh);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_scale_down(lqcd_ctx* c, int dprec, const void* src, void* dst, const double* dscale, double hscale) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(dprec, hipLaunchKernelGGL(k_scale_down<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, src, dst, dscale,
                                           hscale, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_accum_up(lqcd_ctx* c, int sprec, void* x, const void* e, const double* dscale) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(sprec, hipLaunchKernelGGL(k_accum_up<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, x, e, dscale, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_copy(lqcd_ctx* c, int prec, const void* src, void* dst) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_copy<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, src, dst, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_zero(lqcd_ctx* c, int prec, void* dst) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_zero<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, dst, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int blas_scale2(lqcd_ctx* c, int prec, void* p, void* v, double f) {
  const size_t vh = c->g.vh;
  LQ_PREC_SWITCH(prec, hipLaunchKernelGGL(k_scale2<P>, dim3(nblk(vh)), dim3(BS), 0, c->stream, p, v, f, vh));
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int fin_reliable(lqcd_ctx* c, Scal* sc, const double* partials, int n, double target2) {
  hipLaunchKernelGGL(k_fin_reliable, dim3(1), dim3(FBS), 0, c->stream, sc, partials, n, target2);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

int fin_alpha(lqcd_ctx* c, Scal* sc, const double* partials, int n) {
  hipLaunchKernelGGL(k_fin_alpha, dim3(1), dim3(FBS), 0, c->stream, sc, partials, n);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int fin_omega(lqcd_ctx* c, Scal* sc, const double* partials, int n) {
  hipLaunchKernelGGL(k_fin_omega, dim3(1), dim3(FBS), 0, c->stream, sc, partials, n);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int fin_rho(lqcd_ctx* c, Scal* sc, const double* partials, int n) {
  hipLaunchKernelGGL(k_fin_rho, dim3(1), dim3(FBS), 0, c->stream, sc, partials, n);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int fin_init(lqcd_ctx* c, Scal* sc, const double* partials, int n, double target2, int max_iters) {
  hipLaunchKernelGGL(k_fin_init, dim3(1), dim3(FBS), 0, c->stream, sc, partials, n, target2, max_iters);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int fin_norm(lqcd_ctx* c, double* out, const double* partials, int n, int width, int comp) {
  hipLaunchKernelGGL(k_fin_norm, dim3(1), dim3(FBS), 0, c->stream, out, partials, n, width, comp);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

}  // namespace lq
