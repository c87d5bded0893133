// mg_grouped.h -- many independent boxes as grouped level launches.
//
// Boxes of the same grid size and model form a class and run the same cycle
// program, so each level operation of the refined solve (the FP64 outer
// step, the half-sweeps, residual/restriction, coarse source, prolongation,
// the single-workgroup program of the small levels) is one launch per class
// with the box in blockIdx.y: the level kernels keep the register budget and
// the full occupancy of the single-box path, and the launch count no longer
// grows with the number of boxes.  Per-box constants, level geometry and
// workspace pointers come from a table in device memory; a per-box control
// word switches a box off once it has converged or has run its planned
// cycles.  Same per-cell arithmetic as the single-box kernels.
//
// A batch of a few small boxes is bound by issuing launches from one host
// thread (about 4.5 us each): with level operations joined as in the
// single-box path and one reduction, control upload and fork per outer step, 12
// boxes of 32^3-64^3 take 270 launches and 1.9 ms instead of 650 and 3.3.
#pragma once
#include "mg_batched.h"
#include "mg_mid.h"

namespace mgg {

struct GBox {
  int nlev, fused_from;
  int march;           // FP64 outer step by z-marching with two master buffers
  int use_field_in;
  int nbg, nres;       // block partials of kg_pack and of the outer residual
  Lev L[kMaxLevB];
  float h2[kMaxLevB];
  Consts C;
  const float* delta;  // natural n^3
  double* field;       // natural n^3: initial guess (use_field_in) and solution
  float* force;        // natural [3][n^3] or null
  double* w[2];        // FP64 master, packed (w[1]: march only)
  float* e[kMaxLevB];
  float* ea[kMaxLevB];  // colour 1 between a level's way down and up (mg_mid.h)
  float* X[kMaxLevB];
  float* rho[kMaxLevB];
  float* dens[kMaxLevB];
  float* eR[kMaxLevB];
  FusedCorr F;         // levels fused_from .. nlev-1 (the single-workgroup program)
};

// per-box control of the current outer step: cycles to run (kb), whether
// the outer step is taken (on) and the pending correction is to be added;
// corrections added so far once it is (step)
struct GCtl {
  int on, kb, add, step;
};
// pinned host words -> device
__global__ __launch_bounds__(kBlock) void kg_ctl(const GCtl* __restrict__ src,
                                                 GCtl* __restrict__ dst, int nb) {
  for (int q = threadIdx.x; q < nb; q += kBlock) dst[q] = src[q];
}

__device__ __forceinline__ uint32_t gthread() {
  return (uint32_t)blockIdx.x * blockDim.x + threadIdx.x;
}

// natural -> packed density and master; block partials of (bg_coef delta)^2
template <int M>
__global__ __launch_bounds__(kBlock) void kg_pack(const GBox* __restrict__ tab, double* part,
                                                  int pstride) {
  __shared__ double sh[32];
  const GBox& B = tab[blockIdx.y];
  const Lev& L0 = B.L[0];
  const int64_t m = 2 * L0.half;
  const uint32_t g = gthread();
  double t2 = 0.0;
  if (g < (uint32_t)m) {
    int i, j, k;
    dec_nat(g, L0, i, j, k);
    const uint32_t pk = pk_of(L0, i, j, k);
    const float d = B.delta[g];
    B.dens[0][pk] = d;
    if (B.use_field_in) B.w[0][pk] = M == FR ? -B.field[g] : B.field[g];
    else if (!B.march) B.w[0][pk] = B.C.bg;
    const double t = B.C.bg_coef * double(d);
    t2 = t * t;
  }
  const double s = block_sum(t2, sh);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * pstride + blockIdx.x] = s;
}
// the same for march classes (rows of 8 cells, 16-byte aligned inputs): 8
// natural cells per thread.  A box that starts at the uniform background
// leaves its master unwritten (kg_outer_march takes the constant).
template <int M>
__global__ __launch_bounds__(kBlock) void kg_pack8(const GBox* __restrict__ tab, double* part,
                                                   int pstride) {
  __shared__ double sh[32];
  const GBox& B = tab[blockIdx.y];
  const Lev& L0 = B.L[0];
  const uint32_t g8 = gthread();
  double t2 = 0.0;
  if (g8 < (uint32_t)(2 * L0.half / 8)) {
    float v[8];
    ldn<float, 8>(B.delta + (size_t)g8 * 8, v);
    op_pack8<float, float>(L0, v, B.dens[0], 1.0, g8);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double t = B.C.bg_coef * double(v[q]);
      t2 += t * t;
    }
    if (B.use_field_in) {
      double f[8];
      ldn<double, 8>(B.field + (size_t)g8 * 8, f);
      op_pack8<double, double>(L0, f, B.w[0], M == FR ? -1.0 : 1.0, g8);
    }
  }
  const double s = block_sum(t2, sh);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * pstride + blockIdx.x] = s;
}

// density pyramid for the models whose correction operator uses it
__global__ __launch_bounds__(kBlock) void kg_restrict_dens(const GBox* __restrict__ tab, int l) {
  const GBox& B = tab[blockIdx.y];
  const uint32_t g = gthread();
  if (g < (uint32_t)(2 * B.L[l + 1].half))
    op_restrict<float, float>(B.L[l], B.L[l + 1], B.dens[l], B.dens[l + 1], g);
}

// w += e (the pending FP32 correction) where the box takes this outer step
__global__ __launch_bounds__(kBlock) void kg_update(const GBox* __restrict__ tab,
                                                    const GCtl* __restrict__ ctl) {
  const GCtl c = ctl[blockIdx.y];
  if (!c.on || !c.add) return;
  const GBox& B = tab[blockIdx.y];
  const uint32_t g = gthread();
  if (g < (uint32_t)(2 * B.L[0].half)) B.w[0][g] += double(B.e[0][g]);
}

// FP64 residual d = F(w), rho = -d, X = w, e = 0; block partials of d^2
template <int M>
__global__ __launch_bounds__(kBlock) void kg_outer(const GBox* __restrict__ tab,
                                                   const GCtl* __restrict__ ctl, double* part,
                                                   int pstride) {
  __shared__ double sh[32];
  const GCtl c = ctl[blockIdx.y];
  if (!c.on) return;  // uniform over the block: no block_sum below is skipped halfway
  const GBox& B = tab[blockIdx.y];
  const Lev& L0 = B.L[0];
  const uint32_t g = gthread();
  double d = 0.0;
  if (g < (uint32_t)(2 * L0.half)) {
    d = cell_resid_direct<M, double, float>(L0, B.w[0], B.dens[0], (const double*)nullptr, 1.0,
                                            B.C, g);
    B.rho[0][g] = float(-d);
    B.X[0][g] = float(B.w[0][g]);
    B.e[0][g] = 0.0f;
  }
  const double s = block_sum(d * d, sh);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * pstride + blockIdx.x] = s;
}

// The update and the residual in one pass (march classes): w_new = w + e goes
// to the other master buffer while X, rho and the partials are formed, planes
// marching in z.  Memory-bound: 36 bytes a cell against 44 in the two kernels
// above, whose one cell per thread also kept them at 2.6-3.8 TB/s (11 boxes of
// 128^3, other classes running beside: 120 + 214 us, here 116 f(R), 87
// symmetron).  e is left for the next cycle's first half-sweep to overwrite.
template <int M>
__global__ __launch_bounds__(kBlock) void kg_outer_march(const GBox* __restrict__ tab,
                                                         const GCtl* __restrict__ ctl,
                                                         double* part, int pstride, int kt) {
  __shared__ double sh[32];
  const GCtl c = ctl[blockIdx.y];
  if (!c.on) return;
  const GBox& B = tab[blockIdx.y];
  // master before this step's correction; the uniform background as a constant
  const double* src = c.step == 0 ? B.w[0] : B.w[(c.step - 1) & 1];
  if (!B.use_field_in && c.step <= 1) src = nullptr;
  op_outer_fused_kv<M, float, float>(B.L[0], src, c.add ? B.e[0] : (const float*)nullptr,
                                     B.w[c.step & 1], B.dens[0], B.C, B.rho[0], B.X[0],
                                     (float*)nullptr, part + (int64_t)blockIdx.y * pstride,
                                     (double*)nullptr, kt, Store{1, 1, 1, 1}, (double*)nullptr,
                                     sh);
}

// per-box sums of the block partials into pinned host memory, one block per
// box: of the residual (blockIdx.y = 0) and, on the first pass, of the
// background norm (1; its partials follow those of all boxes)
__global__ __launch_bounds__(256) void kg_sum_box(const GBox* __restrict__ tab,
                                                  const double* __restrict__ part, int pstride,
                                                  double* __restrict__ out) {
  __shared__ double sh[32];
  const int bg = blockIdx.y;
  const uint32_t r = bg * gridDim.x + blockIdx.x;
  const int nparts = bg ? tab[blockIdx.x].nbg : tab[blockIdx.x].nres;
  double s = 0.0;
  const double* p = part + (int64_t)r * pstride;
  for (int q = threadIdx.x; q < nparts; q += blockDim.x) s += p[q];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) out[r] = s;
}

// vec: 4 packed cells per thread (the level's rows hold a multiple of 4);
// fresh (vec only): the correction is zero, e uninitialised
template <int M>
__global__ __launch_bounds__(kBlock) void kg_smooth(const GBox* __restrict__ tab,
                                                    const GCtl* __restrict__ ctl, int it, int l,
                                                    int colour, int vec, int fresh) {
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  const Lev& L = B.L[l];
  const uint32_t g = gthread();
  if (vec) {
    if (g < (uint32_t)(L.half / 4))
      op_smooth_corr_v<M>(L, B.e[l], B.X[l], B.dens[l], B.rho[l], colour, B.h2[l], B.C, g, fresh);
  } else if (g < (uint32_t)L.half) {
    op_smooth_corr<M>(L, B.e[l], B.X[l], B.dens[l], B.rho[l], colour, B.h2[l], B.C, g);
  }
}

// the same half-sweep marching in z over kt planes (blocks of one box in x)
template <int M>
__global__ __launch_bounds__(kBlock) void kg_smooth_kv(const GBox* __restrict__ tab,
                                                       const GCtl* __restrict__ ctl, int it, int l,
                                                       int colour, int kt, int fresh) {
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  op_smooth_corr_kv<M, float, float>(B.L[l], B.e[l], B.X[l], B.dens[l], B.rho[l], colour,
                                     B.h2[l], B.C, fresh, kt, Store{1.0f, 1.0f, 1.0f, 1.0f});
}

// residual + restriction of level l in the shifted form (store_coarse_corr):
// the coarse problem is posed around X_H = R X + R e (R X of level l kept in
// eR[l+1], formed again with rx), the coarse correction starts at zero and
// no coarse-source pass follows.
// vec: 4 coarse cells per thread (the coarse side is a multiple of 4);
// zero_e: write the zeros (else the coarse level starts fresh)
template <int M>
__global__ __launch_bounds__(kBlock) void kg_down(const GBox* __restrict__ tab,
                                                  const GCtl* __restrict__ ctl, int it, int l,
                                                  int rx, int skip1, int vec, int zero_e) {
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  const Lev& Lf = B.L[l];
  const Lev& Lc = B.L[l + 1];
  const uint32_t g = gthread();
  float* eH = zero_e ? B.e[l + 1] : nullptr;
  if (vec) {
    if (g < (uint32_t)(2 * Lc.half / 4))
      op_resid_restrict_corr_v<M>(Lf, Lc, B.e[l], B.X[l], B.dens[l], B.rho[l], B.h2[l],
                                  eH, (float*)nullptr, B.rho[l + 1], B.X[l + 1], B.C,
                                  skip1, g, Store{1, 1, 1, 1}, B.eR[l + 1], rx);
  } else if (g < (uint32_t)(2 * Lc.half)) {
    op_resid_restrict_corr<M>(Lf, Lc, B.e[l], B.X[l], B.dens[l], B.rho[l], B.h2[l], eH,
                              (float*)nullptr, B.rho[l + 1], B.X[l + 1], B.C, g, B.eR[l + 1], rx);
  }
}
// e_l += P e_H (the coarse correction of the shifted form); with COL0 = 1
// colour 0 is left to the next exact half-sweep (not for the Newton
// smoother of CQ)
template <int COL0>
__global__ __launch_bounds__(kBlock) void kg_up(const GBox* __restrict__ tab,
                                                const GCtl* __restrict__ ctl, int it, int l) {
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  const uint32_t g = gthread();
  if (g < (uint32_t)(2 * B.L[l + 1].half / 4))
    op_prolong_v<float, COL0>(B.L[l], B.L[l + 1], B.e[l], B.e[l + 1], (const float*)nullptr, g);
}
__global__ __launch_bounds__(kBlock) void kg_up_block(const GBox* __restrict__ tab,
                                                      const GCtl* __restrict__ ctl, int it,
                                                      int l) {
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  const uint32_t g = gthread();
  if (g < (uint32_t)(2 * B.L[l + 1].half))
    op_prolong_block<float>(B.L[l], B.L[l + 1], B.e[l], B.e[l + 1], g);
}

// a level's whole way down and way up in one launch each (mg_mid.h); the boxes
// of a class may differ in the f(R) exponent
template <int M>
__device__ __forceinline__ MidCorr<M, -1, float, float> g_mid_policy(const GBox& B, int l) {
  return {B.X[l], B.rho[l], B.dens[l], B.h2[l], Store{1, 1, 1, 1}, B.C};
}
template <int M>
__global__ __launch_bounds__(kMidThreads) void kg_mid_down(const GBox* __restrict__ tab,
                                                           const GCtl* __restrict__ ctl, int it,
                                                           int l, int rx, int fresh, int zero_e) {
  extern __shared__ __align__(16) unsigned char mid_lds[];
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  mid_down(B.L[l], B.L[l + 1], g_mid_policy<M>(B, l), B.e[l], B.ea[l],
           zero_e ? B.e[l + 1] : nullptr, B.rho[l + 1], B.X[l + 1], B.eR[l + 1], rx, fresh,
           blockIdx.x, reinterpret_cast<float*>(mid_lds));
}
template <int M>
__global__ __launch_bounds__(kMidThreads) void kg_mid_up(const GBox* __restrict__ tab,
                                                         const GCtl* __restrict__ ctl, int it,
                                                         int l) {
  extern __shared__ __align__(16) unsigned char mid_lds[];
  if (it >= ctl[blockIdx.y].kb) return;
  const GBox& B = tab[blockIdx.y];
  mid_up(B.L[l], B.L[l + 1], g_mid_policy<M>(B, l), B.ea[l], B.e[l + 1], B.e[l], blockIdx.x,
         reinterpret_cast<float*>(mid_lds));
}

// the small levels of every box of the class: one workgroup per box
template <int M>
__global__ __launch_bounds__(kFusedThreads) void kg_fused(const GBox* __restrict__ tab,
                                                          const GCtl* __restrict__ ctl, int it,
                                                          FusedProg P) {
  __shared__ double sh[32];
  if (it >= ctl[blockIdx.x].kb) return;
  const GBox& B = tab[blockIdx.x];
  fused_corr_body<M>(B.F, P, B.C, sh);
}

template <int M>
__global__ __launch_bounds__(kFusedThreads) void kg_small(const GBox* __restrict__ tab,
                                                          const GCtl* __restrict__ ctl, int it,
                                                          FusedProg P) {
  extern __shared__ __align__(16) unsigned char small_lds[];
  __shared__ double sh[48];
  if (it >= ctl[blockIdx.x].kb) return;
  const GBox& B = tab[blockIdx.x];
  small_cycle(B.F, P, SmallCorr<M>{B.C}, reinterpret_cast<float*>(small_lds), sh);
}

// packed master -> natural field; kg_unpack8: march classes.  A box stopped
// there before any correction has no master: it is the background.
template <int M>
__global__ __launch_bounds__(kBlock) void kg_unpack(const GBox* __restrict__ tab) {
  const GBox& B = tab[blockIdx.y];
  const Lev& L0 = B.L[0];
  const uint32_t g = gthread();
  if (g >= (uint32_t)(2 * L0.half)) return;
  int i, j, k;
  dec_nat(g, L0, i, j, k);
  const double v = B.w[0][pk_of(L0, i, j, k)];
  B.field[g] = M == FR ? -v : v;
}
template <int M>
__global__ __launch_bounds__(kBlock) void kg_unpack8(const GBox* __restrict__ tab,
                                                     const GCtl* __restrict__ ctl) {
  const GBox& B = tab[blockIdx.y];
  const int step = ctl[blockIdx.y].step;
  const uint32_t g8 = gthread();
  if (g8 >= (uint32_t)(2 * B.L[0].half / 8)) return;
  const double sgn = M == FR ? -1.0 : 1.0;
  if (step == 0 && !B.use_field_in) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = sgn * B.C.bg;
    stn<double, 8>(B.field + (size_t)g8 * 8, v);
  } else {
    op_unpack8<double, double>(B.L[0], B.w[step & 1], B.field, sgn, g8);
  }
}

// fifth force from the natural field, by central differences of Phi5 (the
// products rounded, so equal field values give no force, as in the single-box
// kernels)
template <int M>
__global__ __launch_bounds__(kBlock) void kg_force(const GBox* __restrict__ tab) {
  const GBox& B = tab[blockIdx.y];
  if (!B.force) return;
  const Lev& L0 = B.L[0];
  const int64_t m = 2 * L0.half;
  const uint32_t g = gthread();
  if (g >= (uint32_t)m) return;
  int i, j, k;
  dec_nat(g, L0, i, j, k);
  const int n = L0.n;
  const int ip = i + 1 == n ? 0 : i + 1, im = i == 0 ? n - 1 : i - 1;
  const int jp = j + 1 == n ? 0 : j + 1, jm = j == 0 ? n - 1 : j - 1;
  const int kp = k + 1 == n ? 0 : k + 1, km = k == 0 ? n - 1 : k - 1;
  const double* f = B.field;
  // (f(R): the sign goes with the factor; a negated product would be fused into
  // the difference after all)
  auto phi = [&](double v) {
    return M == SYM ? mul_nc(mul_nc(B.C.phi5, v), v) : mul_nc(B.C.phi5, v);
  };
  const double hm = M == FR ? 0.5 : -0.5;
  const int64_t row = (int64_t)k * n + j;
  B.force[g] = float(hm * (phi(f[row * n + ip]) - phi(f[row * n + im])));
  B.force[m + g] = float(hm * (phi(f[((int64_t)k * n + jp) * n + i]) -
                              phi(f[((int64_t)k * n + jm) * n + i])));
  B.force[2 * m + g] = float(hm * (phi(f[((int64_t)kp * n + j) * n + i]) -
                                  phi(f[((int64_t)km * n + j) * n + i])));
}

}  // namespace mgg
