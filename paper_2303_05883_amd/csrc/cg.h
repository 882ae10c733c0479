// Conjugate gradients with its scalars on the device, shared by the staggered
// and domain-wall solvers: the operator's last launch and the residual update leave
// per-workgroup partial sums, which give alpha, beta and the convergence test, and
// every kernel of an iteration returns at once when the solve is done. Where the
// records are few (fold_ok) the next update adds them itself, each workgroup for
// itself and workgroup 0 writing the state; else a one-block kernel of 4.6 us adds
// them. Per iteration with and without those kernels: staggered 12x10x8x14 FP64 23
// and 26-29 us, 24^3x48 145.6 and 147.5; domain-wall FP32 16^4 x 8 170 and 178. The host only enqueues
// iterations and looks at the state a chunk behind what it has enqueued.
// Against partial sums copied to and added on the host twice per iteration:
// staggered CG on 24^3x48 187 -> 152 us per iteration in FP64 and 128 -> 93 us in
// FP32, on 12x10x8x14 62 -> 32 us; domain-wall FP32 CG on 16^4 x 8 206 -> 179 us.
#pragma once

#include "blas.h"
#include "blascore.h"
#include "internal.h"

namespace lq {

struct CgState {
  double rr[2];    // |r|^2 of the iterated residual before even and odd iterations
  double alpha;
  double beta;
  double target;   // stop when |r| <= target
  int done;        // converged, broken down (<p, A p> not positive) or out of iterations
  int iters;       // iterations done
  int max_iters;
  int last;        // the last iteration to finish, once that is known
};

namespace {

constexpr int CG_FIN = 1024;

// rr from partials (component 1 of the pairs); p = r is set by the caller, so the first beta is 0
__global__ void __launch_bounds__(CG_FIN) k_cg_init(CgState* st, const double* partials, int n, double target,
                                                    int max_iters) {
  double v[2];
  sum_partials<2>(partials, n, v);
  if (threadIdx.x == 0) {
    st->rr[0] = v[1];
    st->alpha = 0.0;
    st->beta = 0.0;
    st->target = target;
    st->iters = 0;
    st->max_iters = max_iters;
    st->done = max_iters <= 0 ? 1 : 0;
    st->last = max_iters <= 0 ? -1 : 0x7fffffff;
  }
}

// Iteration it: alpha = |r|^2 / <p, A p> from the n pairs (component comp); false
// when <p, A p> is not positive, which ends the solve. The writer (one thread of the
// launch) stores them; of what others of the launch read it writes only done, which
// they test by group_flag.
__device__ inline bool cg_alpha_of(CgState* st, const double* partials, int n, int comp, int it, bool writer,
                                   double& alpha) {
  double v[2];
  sum_partials<2>(partials, n, v);
  const double pq = v[comp];
  const bool ok = pq > 0.0;
  alpha = ok ? st->rr[it & 1] / pq : 0.0;
  if (writer) {
    if (ok) {
      st->alpha = alpha;
    } else {
      st->last = it - 1;
      set_flag(&st->done);
    }
  }
  return ok;
}

// The updated |r|^2 (component 1): count, convergence, beta. Workgroups of the same
// launch that start after the writer may see done set: they look at last < it.
__device__ inline double cg_beta_of(CgState* st, const double* partials, int n, int it, bool writer) {
  double v[2];
  sum_partials<2>(partials, n, v);
  const double rn = v[1], beta = rn / st->rr[it & 1];
  if (writer) {
    st->iters = it + 1;
    st->beta = beta;
    st->rr[(it + 1) & 1] = rn;
    if (sqrt(rn) <= st->target || it + 1 >= st->max_iters) {
      st->last = it;
      set_flag(&st->done);
    }
  }
  return beta;
}

__global__ void __launch_bounds__(CG_FIN) k_cg_alpha(CgState* st, const double* partials, int n, int comp, int it) {
  if (st->done) return;
  double alpha;
  cg_alpha_of(st, partials, n, comp, it, threadIdx.x == 0, alpha);
}

__global__ void __launch_bounds__(CG_FIN) k_cg_beta(CgState* st, const double* partials, int n, int it) {
  if (st->done) return;
  cg_beta_of(st, partials, n, it, threadIdx.x == 0);
}

__global__ void __launch_bounds__(CG_FIN) k_cg_sum(double* out, const double* partials, int n) {
  double v[2];
  sum_partials<2>(partials, n, v);
  if (threadIdx.x == 0) {
    out[0] = v[0];
    out[1] = v[1];
  }
}

// This context's state on the device and its two pinned mirrors
inline CgState* cg_state(lqcd_ctx* c) { return reinterpret_cast<CgState*>(c->dscal + 16); }

int cg_init(lqcd_ctx* c, const double* partials, size_t n, double target, int max_iters) {
  hipLaunchKernelGGL(k_cg_init, dim3(1), dim3(CG_FIN), 0, c->stream, cg_state(c), partials, (int)n, target, max_iters);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int cg_alpha(lqcd_ctx* c, const double* partials, size_t n, int comp, int it) {
  hipLaunchKernelGGL(k_cg_alpha, dim3(1), dim3(CG_FIN), 0, c->stream, cg_state(c), partials, (int)n, comp, it);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}
int cg_beta(lqcd_ctx* c, const double* partials, size_t n, int it) {
  hipLaunchKernelGGL(k_cg_beta, dim3(1), dim3(CG_FIN), 0, c->stream, cg_state(c), partials, (int)n, it);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

// The sums of n pairs on the host (blocks)
int cg_sum_host(lqcd_ctx* c, const double* partials, size_t n, double* s0, double* s1) {
  double* d = c->dscal + 32;
  hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(CG_FIN), 0, c->stream, d, partials, (int)n);
  LQ_HIP(hipGetLastError());
  LQ_HIP(hipMemcpyAsync(c->hscal + 32, d, 2 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  LQ_HIP(hipStreamSynchronize(c->stream));
  if (s0) *s0 = c->hscal[32];
  if (s1) *s1 = c->hscal[33];
  return LQCD_OK;
}

// Enqueues iterations (one(it) enqueues iteration it) until the state says done; the host
// waits for the state of one chunk with the next already enqueued. Returns the
// iterations done.
template <typename F>
int cg_run(lqcd_ctx* c, F&& one, int* iters) {
  constexpr int CHUNK = 4;
  struct Events {
    hipEvent_t e[2] = {};
    ~Events() {
      for (auto v : e)
        if (v) (void)hipEventDestroy(v);
    }
  } ev;
  for (auto& e : ev.e) LQ_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  volatile CgState* h[2] = {reinterpret_cast<CgState*>(c->hscal), reinterpret_cast<CgState*>(c->hscal + 16)};
  for (int n = 0, it = 0;; ++n) {
    for (int k = 0; k < CHUNK; ++k, ++it) LQ_TRY(one(it));
    LQ_HIP(hipMemcpyAsync(const_cast<CgState*>(h[n & 1]), cg_state(c), sizeof(CgState), hipMemcpyDeviceToHost, c->stream));
    LQ_HIP(hipEventRecord(ev.e[n & 1], c->stream));
    if (n == 0) continue;
    LQ_HIP(hipEventSynchronize(ev.e[(n - 1) & 1]));
    if (h[(n - 1) & 1]->done) {
      *iters += h[(n - 1) & 1]->iters;
      break;
    }
  }
  LQ_HIP(hipStreamSynchronize(c->stream));  // the last chunk's copy is still to come
  return LQCD_OK;
}

}  // namespace
}  // namespace lq
