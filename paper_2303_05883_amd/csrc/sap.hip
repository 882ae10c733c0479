// Schwarz alternating procedure (SAP) preconditioner and the flexible
// BiCGStab around it (the smoother / preconditioner of the paper's multigrid
// solver, Sec. 3: checkerboard-coloured blocks, the Dirac equation restricted
// to each block with the hops that leave it removed, a fixed number of
// minimal-residual block iterations, the two colours in turn; outer flexible
// BiCGStab).
//
// One workgroup per block of the colour being updated, two lanes per block
// site. The lanes form the block right-hand side rho = eta - D psi at their
// site, then the block's minimal-residual iterations run on chip: the block
// residual sits in LDS, q = D_B r takes its neighbours from LDS and its links
// and clover blocks from registers, the block dot products <q, r> and <q, q> are
// workgroup reductions, and psi += delta goes back to memory.
// The right-hand side is kept up to date instead of recomputed: after a
// colour's update its residual eta - D psi on its own sites is exactly the
// blocks' final MR residual r = rho - D_B delta (the neighbouring blocks are
// of the other colour, so no hop of the update lands on its own colour), and
// the other colour's update changes it only through the hops that cross the
// block faces, by +kappa H delta_other. So each launch stores r and delta, and
// the next launch of the colour starts from r plus those face hops (the
// first launch from eta alone, psi being zero) - no clover term and no
// interior hops from memory.
// The preconditioner works in FP32; the outer solve in FP64.
#include <chrono>
#include <cmath>
#include <cstdio>
#include <vector>

#include "blas.h"
#include "hopcore.h"
#include "internal.h"
#include "ops.h"
#include "sap.h"

namespace lq {
namespace {

struct SapArgs {
  Geom g;
  int b[4];        // block extents
  int nb[4];       // blocks per direction (even)
  int colour;
  int nmr;
  float kappa;
  const char* gauge;  // FP32 links, 2 parities x 4 directions
  size_t link_stride;
  const void* clov[2];  // FP32 A on even / odd sites, or null (Wilson: A = 1)
  const void* base[2];   // eta (first cycle) or the stored block residuals
  const void* dother[2]; // the other colour's last update delta, or null (first launch)
  void* res[2];          // this launch's final block residuals
  void* dout[2];         // this launch's delta
  void* psi[2];
};

__device__ inline void words_put(float4* L, int n, int slot, const cx<float> s[6]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) L[k * n + slot] = make_float4(s[2 * k].r, s[2 * k].i, s[2 * k + 1].r, s[2 * k + 1].i);
}
__device__ inline void words_get(const float4* L, int n, int slot, cx<float> s[6]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float4 v = L[k * n + slot];
    s[2 * k] = {v.x, v.y};
    s[2 * k + 1] = {v.z, v.w};
  }
}

// acc += the forward (sg = 1) or backward (sg = -1) hop in direction MU of the
// neighbour spinor s, m = the matrix to apply (U, or U^dag for a backward hop);
// in t, s[0..5] is the half that survives the projection and lands in the lower
// spins (forward) or the upper ones (backward), and the projection's factor 2 is
// in m.
template <int MU, int HOW>
__device__ inline void pair_hop(const cx<float> s[12], const cx<float> m[9], float sg, cx<float> acc[12]) {
  cx<float> h[6], w[6];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (MU == 0) {  // (1 -+ gamma_mu) psi: h = u +- i sigma l
      h[c] = s[c] + sg * mul_i(s[9 + c]);
      h[3 + c] = s[3 + c] + sg * mul_i(s[6 + c]);
    } else if (MU == 1) {
      h[c] = s[c] + sg * s[9 + c];
      h[3 + c] = s[3 + c] - sg * s[6 + c];
    } else if (MU == 2) {
      h[c] = s[c] + sg * mul_i(s[6 + c]);
      h[3 + c] = s[3 + c] - sg * mul_i(s[9 + c]);
    } else {
      h[c] = s[c];
      h[3 + c] = s[3 + c];
    }
  }
  mat3_mul<true, HOW>(m, h, w);
  const float fw = sg > 0.f ? 1.f : 0.f, bw = 1.f - fw;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cx<float> w0 = w[c], w1 = w[3 + c];
    if (MU == 3) {
      acc[c] = acc[c] + bw * w0;
      acc[3 + c] = acc[3 + c] + bw * w1;
      acc[6 + c] = acc[6 + c] + fw * w0;
      acc[9 + c] = acc[9 + c] + fw * w1;
      continue;
    }
    acc[c] = acc[c] + w0;
    acc[3 + c] = acc[3 + c] + w1;
    if (MU == 0) {  // lower -+= i sigma w
      acc[6 + c] = acc[6 + c] - sg * mul_i(w1);
      acc[9 + c] = acc[9 + c] - sg * mul_i(w0);
    } else if (MU == 1) {
      acc[6 + c] = acc[6 + c] - sg * w1;
      acc[9 + c] = acc[9 + c] + sg * w0;
    } else {
      acc[6 + c] = acc[6 + c] - sg * mul_i(w0);
      acc[9 + c] = acc[9 + c] + sg * mul_i(w1);
    }
  }
}

template <int MU>
__device__ inline void pair_hop_mem(const void* in, size_t j, const cx<float> m[9], float sg,
                                    cx<float> acc[12]) {
  cx<float> s[12];
  if (MU == 3) IO<1>::load_half(in, j, sg < 0.f, s);
  else IO<1>::load_spinor(in, j, s);
  pair_hop<MU, APART>(s, m, sg, acc);
}
// Inside the block the serial multiply-adds: M eta against 64-bit values, 8^4, blocks
// 4^4, 2 cycles of 4 steps, with c_SW 1 and 0, 1.26e-7 and 1.10e-7 (products rounded
// first 1.25e-7 and 1.09e-7, 2-4% slower; one lane per site, products first, kappa on
// every hop 1.44e-7 and 1.22e-7).
template <int MU>
__device__ inline void pair_hop_lds(const float4* Lr, int n, int slot, const cx<float> m[9], float sg,
                                    cx<float> acc[12]) {
  cx<float> s[12];
  if (MU == 3) {
    words_get(sg < 0.f ? Lr : Lr + 3 * n, n, slot, s);
  } else {
    words_get(Lr, n, slot, s);
    words_get(Lr + 3 * n, n, slot, s + 6);
  }
  pair_hop<MU, CHAIN>(s, m, sg, acc);
}

// Each lane of a pair holds a partial sum of all 12 components; the forward lane
// gets the total of the upper spins, the backward lane that of the lower ones.
// v_permlane32_swap exchanges the backward lanes' upper with the forward lanes'
// lower parts.
__device__ inline void pair_total(const cx<float> p[12], cx<float> t[6]) {
  auto one = [](float up, float lo) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, up), __builtin_bit_cast(int, lo), false, false);
    return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
  };
#pragma unroll
  for (int k = 0; k < 6; ++k) t[k] = {one(p[k].r, p[6 + k].r), one(p[k].i, p[6 + k].i)};
}

// Sum of NV doubles over the workgroup, returned to every lane (wave sums, then
// those added in wave order by every lane). A barrier of the caller's stands
// between one use's reads of red and the next use's writes.
template <int NV>
__device__ inline void group_sum(double v[NV], double (*red)[NV]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wave][k] = v[k];
  __syncthreads();
  const int nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w][k];
    v[k] = s;
  }
}

// Two lanes per block site, lanes 0..31 of a wavefront with the forward hops of
// 32 sites and lanes 32..63 with their backward ones: a lane keeps the four
// links it needs (U, or U^dag of the backward neighbours), one chiral block of
// A, and one half (upper or lower spins) of the residual and of delta in
// registers through all block iterations, so an iteration reads nothing but
// the block residual in LDS and has two barriers. Bound by vector issue (about
// 800 instructions per lane and iteration, 230 VGPRs, 2 waves per SIMD), on
// lattices of few blocks by the latency of one block. Against one lane per site
// with the links in LDS and the clover term read again by every iteration (bound
// by latency and those reads), 6 iterations, per launch: 8^3x16 blocks 4x4x2x2
// 52 -> 23 us; 16^3x32 8x4x2x2 65 -> 42 us; 32^3x64 8x4x2x2 770 -> 504 us, 4^4
// 1468 -> 769 us, 16x4x2x2 525 -> 515 us. Held to 128 VGPRs for 4 waves per SIMD
// it spills (813-1227 us for the last). Blocks of fewer than 4 checkerboard
// columns share the cache lines of a row with the next blocks, so these are
// dealt to the XCDs in contiguous ranges (4x4x2x2 on 16^3x32 58 -> 44 us); wider
// ones are not (8x4x2x2 on 32^3x64 533 against 553 us).
__global__ void __launch_bounds__(512) k_sap_block(SapArgs a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ double red[8][3];
  const int n = blockDim.x >> 1;  // block sites
  float4* Lr = reinterpret_cast<float4*>(lds_raw);  // residual, 6 words x n
  const Geom& g = a.g;
  // the blockIdx-th block of this colour: rows of nb[0] blocks alternate colours
  const int hx = a.nb[0] / 2;
  const int lb = logical_block(a.b[0] < 8);
  const int q = lb % hx, row = lb / hx;
  const int by = row % a.nb[1], bz = (row / a.nb[1]) % a.nb[2], bt = row / (a.nb[1] * a.nb[2]);
  const int bx = 2 * q + ((by + bz + bt + a.colour) & 1);
  // this lane's site and side
  const int h = (threadIdx.x >> 5) & 1;
  const bool fwd = h == 0;
  const float sg = fwd ? 1.f : -1.f;
  const int l = ((threadIdx.x >> 6) << 5) | (threadIdx.x & 31);
  const int lx = l % a.b[0], ly = (l / a.b[0]) % a.b[1], lz = (l / (a.b[0] * a.b[1])) % a.b[2],
            lt = l / (a.b[0] * a.b[1] * a.b[2]);
  const int x = bx * a.b[0] + lx, y = by * a.b[1] + ly, z = bz * a.b[2] + lz, t = bt * a.b[3] + lt;
  const int p = (x + y + z + t) & 1;
  const int lxh = g.lxh;
  auto hidx = [&](int xx, int yy, int zz, int tt) -> size_t {
    return (size_t)(xx >> 1) + (size_t)lxh * (yy + (size_t)g.ly * (zz + (size_t)g.lz * tt));
  };
  const size_t i = hidx(x, y, z, t);
  const size_t ls = a.link_stride;
  const char* gl = a.gauge + (size_t)((fwd ? p : 1 - p) * 4) * ls;  // forward links here, backward ones at x - mu
  const int c[4] = {x, y, z, t}, L[4] = {g.lx, g.ly, g.lz, g.lt};
  const int lc[4] = {lx, ly, lz, lt};
  const int stride[4] = {1, a.b[0], a.b[0] * a.b[1], a.b[0] * a.b[1] * a.b[2]};
  bool in_block[4];  // the neighbour on this lane's side is in the block
  size_t j[4];       // its checkerboard index
  int slot[4];
  cx<float> m[4][9];  // the matrix of this lane's hop in direction mu
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    in_block[mu] = fwd ? lc[mu] + 1 < a.b[mu] : lc[mu] > 0;
    slot[mu] = fwd ? l + stride[mu] : l - stride[mu];
    int d[4] = {c[0], c[1], c[2], c[3]};
    d[mu] = fwd ? (c[mu] + 1 == L[mu] ? 0 : c[mu] + 1) : (c[mu] == 0 ? L[mu] - 1 : c[mu] - 1);
    j[mu] = hidx(d[0], d[1], d[2], d[3]);
    cx<float> u[6], r2[3];
    IO<1>::template load_link<false>(gl + mu * ls, fwd ? i : j[mu], u);
    reconstruct(u, r2);
    // 2 for the t projection and the boundary factor of a hop that crosses the
    // lattice (never inside a block) are folded in, both exact in FP32; kappa,
    // which would round every element, multiplies the sum of the hops instead
    const bool wrap = mu == 3 && g.t_bc < 0 && (fwd ? t + 1 == L[3] : t == 0);
    const float f = (mu == 3 ? 2.f : 1.f) * (wrap ? -1.f : 1.f);
    const cx<float> u9[9] = {u[0], u[1], u[2], u[3], u[4], u[5], r2[0], r2[1], r2[2]};
#pragma unroll
    for (int k = 0; k < 9; ++k) m[mu][k] = f * (fwd ? u9[k] : conj(u9[3 * (k % 3) + k / 3]));
  }

  // ---- rho = base + kappa (H delta_other) over the hops that cross the block
  // faces (neighbours from memory; the interior hops are in base)
  cx<float> acc[12], r[6];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = {0.f, 0.f};
  if (a.dother[1 - p]) {
    const void* pin = a.dother[1 - p];
    if (!in_block[0]) pair_hop_mem<0>(pin, j[0], m[0], sg, acc);
    if (!in_block[1]) pair_hop_mem<1>(pin, j[1], m[1], sg, acc);
    if (!in_block[2]) pair_hop_mem<2>(pin, j[2], m[2], sg, acc);
    if (!in_block[3]) pair_hop_mem<3>(pin, j[3], m[3], sg, acc);
  }
  {
    cx<float> hop[6];
    pair_total(acc, hop);
    IO<1>::load_half(a.base[p], i, fwd, r);
#pragma unroll
    for (int k = 0; k < 6; ++k) r[k] = caxpy(a.kappa, hop[k], r[k]);
  }
  const bool clover = a.clov[0] != nullptr;
  cx<float> cb[18];
  if (clover) IO<1>::template load_clover_block<false>(a.clov[p], i, h, cb);

  cx<float> ps[6];  // read early, added to at the end
  IO<1>::load_half(a.psi[p], i, fwd, ps);

  // ---- minimal-residual iterations on the block
  cx<float> delta[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) delta[k] = {0.f, 0.f};
  for (int it = 0; it < a.nmr; ++it) {
    // the previous residual has been read: every wave has passed the barrier of
    // the sums since
    words_put(Lr + 3 * h * n, n, l, r);
    __syncthreads();
    // q = D_B r = A r - kappa sum of the hops that stay in the block
    cx<float> qv[12], qh[6];
#pragma unroll
    for (int k = 0; k < 12; ++k) qv[k] = {0.f, 0.f};
    if (in_block[0]) pair_hop_lds<0>(Lr, n, slot[0], m[0], sg, qv);
    if (in_block[1]) pair_hop_lds<1>(Lr, n, slot[1], m[1], sg, qv);
    if (in_block[2]) pair_hop_lds<2>(Lr, n, slot[2], m[2], sg, qv);
    if (in_block[3]) pair_hop_lds<3>(Lr, n, slot[3], m[3], sg, qv);
    if (clover) {
      // this lane's chiral block: c_+- = u -+ l, A c added to (u, l) as (y, -+ y)
      cx<float> o[6], ch[6], yv[6];
      words_get(Lr + 3 * (1 - h) * n, n, l, o);
#pragma unroll
      for (int k = 0; k < 6; ++k) ch[k] = fwd ? r[k] - o[k] : o[k] + r[k];
      herm6_mul(cb, ch, yv);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        qv[k] = caxpy(-a.kappa, qv[k], yv[k]);
        qv[6 + k] = caxpy(-a.kappa, qv[6 + k], -sg * yv[k]);
      }
    }
    pair_total(qv, qh);
    if (!clover)
#pragma unroll
      for (int k = 0; k < 6; ++k) qh[k] = caxpy(-a.kappa, qh[k], r[k]);
    double dv[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const cx<float> d = cmulc(qh[k], r[k]);
      dv[0] += (double)d.r;
      dv[1] += (double)d.i;
      dv[2] += (double)qh[k].r * qh[k].r + (double)qh[k].i * qh[k].i;
    }
    group_sum<3>(dv, red);
    const cx<float> alpha = dv[2] > 0.0 ? cx<float>{(float)(dv[0] / dv[2]), (float)(dv[1] / dv[2])}
                                        : cx<float>{0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      delta[k] = delta[k] + alpha * r[k];
      r[k] = r[k] - alpha * qh[k];
    }
  }
  // ---- psi += delta on this block; the residual and delta for the next launches
  auto store_half = [&](void* f, const cx<float> s[6]) {
    float4* o = reinterpret_cast<float4*>(f);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      o[widx(i, 3 * h + k, 6)] = make_float4(s[2 * k].r, s[2 * k].i, s[2 * k + 1].r, s[2 * k + 1].i);
  };
  store_half(a.res[p], r);
  store_half(a.dout[p], delta);
#pragma unroll
  for (int k = 0; k < 6; ++k) ps[k] = ps[k] + delta[k];
  store_half(a.psi[p], ps);
}

}  // namespace

bool sap_shape_ok(const Geom& g, const int b[4]) {
  const int L[4] = {g.lx, g.ly, g.lz, g.lt};
  int vol = 1;
  for (int d = 0; d < 4; ++d) {
    if (b[d] < 1 || L[d] % b[d] != 0 || (L[d] / b[d]) % 2 != 0) return false;
    vol *= b[d];
  }
  return vol >= 64 && vol <= 256 && vol % 64 == 0;
}

// psi = M eta on FP32 native half fields (eta, psi: even and odd halves).
int sap_apply(lqcd_ctx* c, const int b[4], int ncy, int nmr, const void* eta_e, const void* eta_o, void* psi_e,
              void* psi_o) {
  if (!sap_shape_ok(c->g, b)) return set_error(LQCD_EINVAL, "bad SAP block shape");
  if (ncy < 1 || nmr < 1) return set_error(LQCD_EINVAL, "SAP needs at least one cycle and one block iteration");
  SapArgs a{};
  a.g = c->g;
  const int L[4] = {c->g.lx, c->g.ly, c->g.lz, c->g.lt};
  int vol = 1, nblocks = 1;
  for (int d = 0; d < 4; ++d) {
    a.b[d] = b[d];
    a.nb[d] = L[d] / b[d];
    vol *= b[d];
    nblocks *= a.nb[d];
  }
  a.nmr = nmr;
  a.kappa = (float)c->kappa;
  a.gauge = reinterpret_cast<const char*>(c->gauge[1]);
  a.link_stride = link_bytes(1, c->g.vh);
  a.clov[0] = clover_slot(c, 1, 0);
  a.clov[1] = clover_slot(c, 1, 1);
  const size_t hb = spinor_bytes(1, c->g.vh);
  for (void** f : {&c->sap_res, &c->sap_delta})
    if (!*f) LQ_TRY(device_alloc(f, 2 * hb, "SAP workspace allocation failed"));
  char* res = static_cast<char*>(c->sap_res);
  char* del = static_cast<char*>(c->sap_delta);
  a.psi[0] = psi_e;
  a.psi[1] = psi_o;
  a.res[0] = res;
  a.res[1] = res + hb;
  a.dout[0] = del;
  a.dout[1] = del + hb;
  LQ_TRY(blas_zero(c, 1, psi_e));
  LQ_TRY(blas_zero(c, 1, psi_o));
  const size_t lds = (size_t)vol * 6 * 16;
  for (int cy = 0; cy < ncy; ++cy)
    for (int colour = 0; colour < 2; ++colour) {
      a.colour = colour;
      // right-hand side: eta on the first cycle, then this colour's stored
      // residual; plus the face hops of the other colour's last update (none
      // before the first update)
      a.base[0] = cy == 0 ? eta_e : res;
      a.base[1] = cy == 0 ? eta_o : res + hb;
      const bool none = cy == 0 && colour == 0;
      a.dother[0] = none ? nullptr : del;
      a.dother[1] = none ? nullptr : del + hb;
      hipLaunchKernelGGL(k_sap_block, dim3(nblocks / 2), dim3(2 * vol), lds, c->stream, a);
    }
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

}  // namespace lq

// ------------------------------------------------------------------ flexible BiCGStab (FP64)
namespace lq {
namespace {

constexpr int LBS = 256;

// out = ca a + cb b + cc c on FP64 half fields (b, c may be null)
__global__ void __launch_bounds__(LBS) k_lin3(void* out, const void* a, cx<double> ca, const void* b, cx<double> cb,
                                              const void* cc_f, cx<double> cc, size_t vh) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= vh) return;
  cx<double> va[12], w[12];
  IO<0>::load_spinor(a, i, va);
#pragma unroll
  for (int k = 0; k < 12; ++k) w[k] = ca * va[k];
  if (b) {
    IO<0>::load_spinor(b, i, va);
#pragma unroll
    for (int k = 0; k < 12; ++k) w[k] = w[k] + cb * va[k];
  }
  if (cc_f) {
    IO<0>::load_spinor(cc_f, i, va);
#pragma unroll
    for (int k = 0; k < 12; ++k) w[k] = w[k] + cc * va[k];
  }
  IO<0>::store_spinor(out, i, w);
}

// per-workgroup partial sums of <a, b> (re, im) and <b, b> on FP64 half fields
__global__ void __launch_bounds__(LBS) k_dot(const void* a, const void* b, double* partials, size_t vh) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  double v[3] = {0.0, 0.0, 0.0};
  if (i < vh) {
    cx<double> x[12], y[12];
    IO<0>::load_spinor(a, i, x);
    IO<0>::load_spinor(b, i, y);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const cx<double> d = cmulc(x[k], y[k]);
      v[0] += d.r;
      v[1] += d.i;
      v[2] += y[k].r * y[k].r + y[k].i * y[k].i;
    }
  }
  block_reduce<3>(v, partials + (size_t)blockIdx.x * 3);
}

struct Pair {
  void* h[2] = {nullptr, nullptr};
};

struct FWork {
  Scratch mem;
  double* partials = nullptr;
  std::vector<double> host;
  explicit FWork(lqcd_ctx* c) : mem(c) {}
  int alloc(size_t bytes, void** p) { return mem.get(bytes, p, "SAP solver workspace allocation failed"); }
};

int grid_of(size_t n) { return (int)((n + LBS - 1) / LBS); }

int lin3(lqcd_ctx* c, Pair out, cx<double> ca, Pair a, cx<double> cb = {0, 0}, const Pair* b = nullptr,
         cx<double> cc = {0, 0}, const Pair* cf = nullptr) {
  const size_t vh = c->g.vh;
  for (int h = 0; h < 2; ++h)
    hipLaunchKernelGGL(k_lin3, dim3(grid_of(vh)), dim3(LBS), 0, c->stream, out.h[h], a.h[h], ca, b ? b->h[h] : nullptr,
                       cb, cf ? cf->h[h] : nullptr, cc, vh);
  LQ_HIP(hipGetLastError());
  return LQCD_OK;
}

// <a, b> and ||b||^2 over both halves, summed on the host in a fixed order
int dot(lqcd_ctx* c, FWork& w, Pair a, Pair b, cx<double>* ab, double* bb) {
  const size_t vh = c->g.vh;
  const int nb = grid_of(vh);
  for (int h = 0; h < 2; ++h)
    hipLaunchKernelGGL(k_dot, dim3(nb), dim3(LBS), 0, c->stream, a.h[h], b.h[h], w.partials + (size_t)h * nb * 3, vh);
  LQ_HIP(hipGetLastError());
  w.host.resize((size_t)2 * nb * 3);
  LQ_HIP(hipMemcpyAsync(w.host.data(), w.partials, w.host.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  LQ_HIP(hipStreamSynchronize(c->stream));
  double s[3] = {0.0, 0.0, 0.0};
  for (size_t k = 0; k < w.host.size(); k += 3)
    for (int j = 0; j < 3; ++j) s[j] += w.host[k + j];
  if (ab) *ab = {s[0], s[1]};
  if (bb) *bb = s[2];
  return LQCD_OK;
}

inline cx<double> cdivd(cx<double> a, cx<double> b) {
  const double d = b.r * b.r + b.i * b.i;
  return {(a.r * b.r + a.i * b.i) / d, (a.i * b.r - a.r * b.i) / d};
}

}  // namespace

// D x = b on the full lattice (FP64 native halves) by flexible BiCGStab with
// the preconditioner pre on the right (FP64 halves in, FP64 halves out; it may
// vary between calls); stops on the true residual. name labels the log lines.
int solve_flexible(lqcd_ctx* c, const lqcd_solve_params& prm, const FlexPrecond& pre, const char* name,
                   const void* b_e, const void* b_o, void* x_e, void* x_o, bool zero_x, lqcd_solve_stats& st) {
  using clk = std::chrono::steady_clock;
  const auto t0 = clk::now();
  FWork w(c);
  const size_t b64 = spinor_bytes(0, c->g.vh);
  Pair r, rh, p, v, s, t, ph, sh, ax;
  for (Pair* q : {&r, &rh, &p, &v, &s, &t, &ax})
    for (auto& h : q->h) LQ_TRY(w.alloc(b64, &h));
  // without a preconditioner (plain BiCGStab) the preconditioned vectors are
  // the vectors themselves: p_hat aliases p and s_hat aliases s
  const bool ident = !pre;
  if (ident) {
    ph = p;
    sh = s;
  } else {
    for (Pair* q : {&ph, &sh})
      for (auto& h : q->h) LQ_TRY(w.alloc(b64, &h));
  }
  LQ_TRY(w.alloc((size_t)2 * grid_of(c->g.vh) * 3 * sizeof(double), reinterpret_cast<void**>(&w.partials)));
  Pair b, x;
  b.h[0] = const_cast<void*>(b_e);
  b.h[1] = const_cast<void*>(b_o);
  x.h[0] = x_e;
  x.h[1] = x_o;
  if (zero_x) {
    LQ_TRY(blas_zero(c, 0, x_e));
    LQ_TRY(blas_zero(c, 0, x_o));
  }
  auto apply = [&](Pair in, Pair out) -> int { return op_full(c, 0, in.h[0], in.h[1], out.h[0], out.h[1]); };
  int napply = 0;
  auto precond = [&](Pair in, Pair out) -> int {
    if (ident) return LQCD_OK;
    LQ_TRY(pre(in.h[0], in.h[1], out.h[0], out.h[1]));
    ++napply;
    return LQCD_OK;
  };
  double bb = 0.0;
  LQ_TRY(dot(c, w, b, b, nullptr, &bb));
  const double bnorm = std::sqrt(bb);
  st = lqcd_solve_stats{};
  const auto t1 = clk::now();
  st.seconds_setup = std::chrono::duration<double>(t1 - t0).count();
  if (bnorm == 0.0) {
    LQ_TRY(blas_zero(c, 0, x_e));
    LQ_TRY(blas_zero(c, 0, x_o));
    st.true_rel_resid = 0.0;
    return LQCD_OK;
  }
  const double target = prm.tol * bnorm;
  int iters = 0, restarts = 0, status = LQCD_OK;
  double rnorm = 0.0;
  for (;;) {
    // true residual r = b - D x
    LQ_TRY(apply(x, ax));
    LQ_TRY(lin3(c, r, {1, 0}, b, {-1, 0}, &ax));
    double rr = 0.0;
    LQ_TRY(dot(c, w, r, r, nullptr, &rr));
    rnorm = std::sqrt(rr);
    if (log_level() >= 1)
      std::fprintf(stderr, "[lqcd] %s-FBiCGStab restart %d: %d iterations, |r|/|b| %.3e\n", name, restarts, iters,
                   rnorm / bnorm);
    if (rnorm <= target) break;
    if (!(rnorm == rnorm)) {
      status = set_error(LQCD_EBREAKDOWN, "preconditioned flexible BiCGStab produced NaN");
      break;
    }
    if (iters >= prm.max_iter || restarts > prm.max_outer) {
      status = set_error(LQCD_ENOCONV, "preconditioned flexible BiCGStab did not reach the tolerance");
      break;
    }
    LQ_TRY(lin3(c, rh, {1, 0}, r));
    cx<double> rho_old{1, 0}, alpha{1, 0}, omega{1, 0};
    LQ_TRY(blas_zero(c, 0, v.h[0]));
    LQ_TRY(blas_zero(c, 0, v.h[1]));
    LQ_TRY(blas_zero(c, 0, p.h[0]));
    LQ_TRY(blas_zero(c, 0, p.h[1]));
    // rho = <rhat, r>; later iterations take it from the residual-norm pass
    cx<double> rho;
    LQ_TRY(dot(c, w, rh, r, &rho, nullptr));
    while (iters < prm.max_iter) {
      if (rho.r == 0.0 && rho.i == 0.0) break;
      const cx<double> beta = cdivd(rho, rho_old) * cdivd(alpha, omega);
      // p = r + beta (p - omega v)
      LQ_TRY(lin3(c, p, {1, 0}, r, beta, &p, {-(beta * omega).r, -(beta * omega).i}, &v));
      LQ_TRY(precond(p, ph));
      LQ_TRY(apply(ph, v));
      cx<double> rv;
      LQ_TRY(dot(c, w, rh, v, &rv, nullptr));
      if (rv.r == 0.0 && rv.i == 0.0) break;
      alpha = cdivd(rho, rv);
      LQ_TRY(lin3(c, s, {1, 0}, r, {-alpha.r, -alpha.i}, &v));
      LQ_TRY(precond(s, sh));
      LQ_TRY(apply(sh, t));
      // one pass: <s, t> (its conjugate is <t, s>) and <t, t>
      cx<double> st;
      double tt = 0.0;
      LQ_TRY(dot(c, w, s, t, &st, &tt));
      omega = tt != 0.0 ? cx<double>{st.r / tt, -st.i / tt} : cx<double>{0, 0};
      LQ_TRY(lin3(c, x, {1, 0}, x, alpha, &ph, omega, &sh));
      LQ_TRY(lin3(c, r, {1, 0}, s, {-omega.r, -omega.i}, &t));
      rho_old = rho;
      ++iters;
      // one pass: the next rho = <rhat, r> and |r|^2
      double rn2 = 0.0;
      LQ_TRY(dot(c, w, rh, r, &rho, &rn2));
      if (log_level() >= 2)
        std::fprintf(stderr, "[lqcd] %s-FBiCGStab iteration %d: |r|/|b| %.3e\n", name, iters, std::sqrt(rn2) / bnorm);
      if (std::sqrt(rn2) <= target || (omega.r == 0.0 && omega.i == 0.0)) break;
    }
    ++restarts;
  }
  st.outer_iters = iters;
  st.inner_iters = napply;
  st.restarts = restarts > 0 ? restarts - 1 : 0;
  st.true_rel_resid = rnorm / bnorm;
  st.seconds_solve = std::chrono::duration<double>(clk::now() - t1).count();
  return status;
}

// D x = b with FP64 flexible BiCGStab, the FP32 SAP preconditioner on the right.
int solve_sap(lqcd_ctx* c, const lqcd_solve_params& prm, const int blk[4], int ncy, int nmr, const void* b_e,
              const void* b_o, void* x_e, void* x_o, bool zero_x, lqcd_solve_stats& st) {
  if (!sap_shape_ok(c->g, blk)) return set_error(LQCD_EINVAL, "bad SAP block shape");
  const size_t b32 = spinor_bytes(1, c->g.vh);
  FWork w(c);
  Pair e32, q32;
  for (Pair* q : {&e32, &q32})
    for (auto& h : q->h) LQ_TRY(w.alloc(b32, &h));
  FlexPrecond pre = [&](const void* ie, const void* io, void* oe, void* oo) -> int {
    LQ_TRY(launch_convert_field(c, 0, ie, 1, e32.h[0]));
    LQ_TRY(launch_convert_field(c, 0, io, 1, e32.h[1]));
    LQ_TRY(sap_apply(c, blk, ncy, nmr, e32.h[0], e32.h[1], q32.h[0], q32.h[1]));
    LQ_TRY(launch_convert_field(c, 1, q32.h[0], 0, oe));
    LQ_TRY(launch_convert_field(c, 1, q32.h[1], 0, oo));
    return LQCD_OK;
  };
  return solve_flexible(c, prm, pre, "SAP", b_e, b_o, x_e, x_o, zero_x, st);
}

}  // namespace lq
