// mg_mid.h -- whole descents and ascents of one middle level in one launch.
//
// On levels of a few 10^4 to 10^5 cells a half-sweep, a restriction or a
// prolongation takes 4-8 us, nearly all of it the launch and the latency of one
// dependent pass over data that lie in cache.  The two kernels here run the
// level's way down (colour-0 and colour-1 half-sweep, residual, restriction)
// and its way up (prolongation, both half-sweeps) in one launch each: a
// workgroup owns kMidT x kMidT fine rows (whole rows: x is periodic inside
// the tile), recomputes what it needs of the rows around them (down: colour 0
// up to two rows away, colour 1 one row away; up: the prolonged colour 1 two
// rows away, colour 0 one row away) and passes values between the half-sweeps
// through LDS.  Rows further than that in j and k together are left out.  For
// smoothers that solve each cell exactly (f(R), symmetron, the linear
// operator): colour 0 need not be kept between the two, and colour 1 goes
// through a buffer of its own, since neighbouring workgroups still read the
// values it replaces.  Per-cell arithmetic and summation orders are those of the
// kernels they replace (bit-identical).
//
// Down / up take 5.0 / 4.8 us at 32^3 (f(R); 256 threads: 7.6 / 6.5) against 17 /
// 15 for the separate kernels and 7.3 / 7.1 against 18 / 16 at 64^3 (symmetron),
// where the launch and four dependent phases bound them.  Recomputation makes the
// way down solve 52 + 32 rows of cells for its 16 + 16 (2.6 times), the way up
// 32 + 16 (1.5 times) after prolonging 52 rows for 16 (3.25 times), and from 96^3
// on that eats the gain (96^3: 22 / 20 against 21 / 19 us, 128^3: 30 / 31 against
// 26 / 22), so the kernels are used up to kMidMaxN cells a side.
#pragma once
#include "mg_kernels.h"

namespace mgg {

constexpr int kMidT = 4;             // fine rows per tile in j and in k
constexpr int kMidS = kMidT + 4;     // with two rows around
constexpr int kMidThreads = 1024;
constexpr int kMidMaxN = 80;
constexpr int kMidSC = kMidT / 2 + 4;  // coarse rows per tile side of the way up

// Correction form: cell data of a level in its storage
template <int M, int N, typename TX, typename TR>
struct MidCorr {
  static_assert(M != CQ, "the smoother solves each cell exactly");
  static constexpr bool kShift = true;  // coarse problem around R X + R e
  const TX* X;
  const TR* rho;
  const float* dens;
  float h2;
  Store S;
  Consts C;
  struct Cell {
    float x, r, d;
  };
  template <typename TS>
  __device__ __forceinline__ static float dec1(TS v, float dec) {
    if constexpr (sizeof(TS) == 4) return v;
    else return mul_nc(float(v), dec);
  }
  __device__ __forceinline__ Cell load(uint32_t q) const {
    return Cell{dec1(X[q], S.x_dec), dec1(rho[q], S.r_dec), M == FR ? 0.0f : dens[q]};
  }
  __device__ __forceinline__ float update(const Cell& c, float sum) const {
    return corr_update<M>(with_exponent<M, N>(C), h2, 0.0f, sum, c.x, c.d, c.r);
  }
  __device__ __forceinline__ float resid(const Cell& c, float u, float sum) const {
    return corr_G<M>(with_exponent<M, N>(C), h2, u, sum, c.x, c.d) - c.r;
  }
  // sx += X of a cell of colour 0 (decoded, then added) or 1 (one rounding)
  __device__ __forceinline__ float add_x(uint32_t q, int colour, float sx) const {
    if constexpr (sizeof(TX) == 4) return sx + X[q];
    else return colour ? __fmaf_rn(float(X[q]), S.x_dec, sx) : sx + mul_nc(float(X[q]), S.x_dec);
  }
};
// Linear operator (adjoint): A v = kap (6 v - sum)/h^2 + dg v, kh2 = kap/h^2
// quads: as the kernels on rows of a multiple of 4 cells (lin_cell_f), else as
// the per-cell ones
template <typename TD, typename TR>
struct MidLin {
  static constexpr bool kShift = false;
  const TD* dg;
  const TR* r;
  float kh2;
  Store S;
  int quads;
  struct Cell {
    float d, r;
  };
  template <typename TS>
  __device__ __forceinline__ static float dec1(TS v, float dec) {
    if constexpr (sizeof(TS) == 4) return v;
    else return mul_nc(float(v), dec);
  }
  __device__ __forceinline__ Cell load(uint32_t q) const {
    return Cell{dec1(dg[q], S.x_dec), dec1(r[q], S.r_dec)};
  }
  __device__ __forceinline__ float update(const Cell& c, float sum) const {
    if (quads) return lin_cell_f(c.r, sum, c.d, kh2);
    return (c.r + kh2 * sum) / (6.0f * kh2 + c.d);
  }
  __device__ __forceinline__ float resid(const Cell& c, float u, float sum) const {
    return c.r - (kh2 * (6.0f * u - sum) + c.d * u);
  }
  __device__ __forceinline__ float add_x(uint32_t, int, float sx) const { return sx; }
};

// Row of a tile: place in the kMidS x kMidS frame, distance from the owned
// rows (|dj| + |dk| outside them) and the level's row.
struct MidRow {
  int rj, rk, dist, j, k;
};
__device__ __forceinline__ MidRow mid_row(int row, int j0, int k0, int n) {
  MidRow r;
  r.rj = row % kMidS;
  r.rk = row / kMidS;
  const int dj = r.rj < 2 ? 2 - r.rj : (r.rj > kMidT + 1 ? r.rj - kMidT - 1 : 0);
  const int dk = r.rk < 2 ? 2 - r.rk : (r.rk > kMidT + 1 ? r.rk - kMidT - 1 : 0);
  r.dist = dj + dk;
  r.j = j0 + r.rj - 2;
  r.j = r.j < 0 ? r.j + n : (r.j >= n ? r.j - n : r.j);
  r.k = k0 + r.rk - 2;
  r.k = r.k < 0 ? r.k + n : (r.k >= n ? r.k - n : r.k);
  return r;
}
// neighbour sum (nbsum's order) of cell ih of the colour in tile row (rj, rk)
// from the other colour's rows o in LDS
__device__ __forceinline__ float mid_sum(const float* o, int row, int ih, int nh, int s) {
  const float* c = o + row * nh;
  const int xe = s ? (ih + 1 == nh ? 0 : ih + 1) : (ih == 0 ? nh - 1 : ih - 1);
  return (c[ih] + c[xe]) + (c[ih - nh] + c[ih + nh]) + (c[ih - kMidS * nh] + c[ih + kMidS * nh]);
}

__host__ inline size_t mid_down_lds(const Lev& Lf) {
  return sizeof(float) * (size_t)Lf.nh * (2 * kMidS * kMidS + 2 * kMidT * kMidT);
}
__host__ inline size_t mid_up_lds(const Lev& Lf) {
  return sizeof(float) * (size_t)Lf.nh * (2 * kMidS * kMidS + kMidSC * kMidSC);
}
__host__ inline unsigned mid_blocks(const Lev& Lf) {
  return (unsigned)(Lf.n / kMidT) * (unsigned)(Lf.n / kMidT);
}

// The way down.  e: the level's correction (read where not fresh), ea: its
// colour 1 after the sweep (n^3/2 values); coarse outputs as
// store_coarse_corr's shifted form (kShift) or rhoH = R(r - A e), eH = 0.
// Colour 1, swept last, has zero residual, which is left out on rows of a
// multiple of 4 cells and computed (rounding noise) on others, as the separate
// kernels do.
template <class P>
__device__ __forceinline__ void mid_down(const Lev& Lf, const Lev& Lc, const P& p,
                                         const float* __restrict__ e, float* __restrict__ ea,
                                         float* eH, float* rhoH, float* XH, float* Xf, int rx,
                                         int fresh, uint32_t tile, float* lds) {
  const int n = Lf.n, nh = Lf.nh, nt = n / kMidT;
  const uint32_t half = (uint32_t)Lf.half;
  const int tk = (int)tile / nt, j0 = ((int)tile - tk * nt) * kMidT, k0 = tk * kMidT;
  float* E0 = lds;
  float* E1 = E0 + kMidS * kMidS * nh;
  float* Z = E1 + kMidS * kMidS * nh;  // residuals of the owned cells
  const int own_cells = kMidT * kMidT * nh;
  const bool both = nh % 4 != 0;
  const int all = kMidS * kMidS * nh;
  for (int g = threadIdx.x; g < all; g += kMidThreads) {
    const int row = (int)Lf.dnh.div((uint32_t)g), ih = g - row * nh;
    const MidRow r = mid_row(row, j0, k0, n);
    if (r.dist > 2) continue;
    const uint32_t q = prow(Lf, r.j, r.k) + (uint32_t)ih;
    const float sum =
        fresh ? 0.0f : nbsum<float>(Lf, e + half, ih, r.j, r.k, (r.j + r.k) & 1);
    E0[g] = p.update(p.load(q), sum);
  }
  __syncthreads();
  for (int g = threadIdx.x; g < all; g += kMidThreads) {
    const int row = (int)Lf.dnh.div((uint32_t)g), ih = g - row * nh;
    const MidRow r = mid_row(row, j0, k0, n);
    if (r.dist > 1) continue;
    const uint32_t q = prow(Lf, r.j, r.k) + (uint32_t)ih;
    const float v = p.update(p.load(half + q), mid_sum(E0, row, ih, nh, (r.j + r.k + 1) & 1));
    E1[g] = v;
    if (r.dist == 0) ea[q] = v;
  }
  __syncthreads();
  for (int g = threadIdx.x; g < own_cells; g += kMidThreads) {
    const int own = (int)Lf.dnh.div((uint32_t)g), ih = g - own * nh;
    const int j = j0 + own % kMidT, k = k0 + own / kMidT;
    const int row = (own / kMidT + 2) * kMidS + own % kMidT + 2;
    const uint32_t q = prow(Lf, j, k) + (uint32_t)ih;
    Z[g] = p.resid(p.load(q), E0[row * nh + ih], mid_sum(E1, row, ih, nh, (j + k) & 1));
    if (both)
      Z[own_cells + g] = p.resid(p.load(half + q), E1[row * nh + ih],
                                 mid_sum(E0, row, ih, nh, (j + k + 1) & 1));
  }
  __syncthreads();
  const bool want_x = P::kShift && rx;
  for (int g = threadIdx.x; g < (kMidT / 2) * (kMidT / 2) * nh; g += kMidThreads) {
    const int own = (int)Lf.dnh.div((uint32_t)g), I = g - own * nh;
    const int cj = own % (kMidT / 2), ck = own / (kMidT / 2);
    float se = 0.0f, sd = 0.0f, sx = 0.0f;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int lj = 2 * cj + b, lk = 2 * ck + d;
        const int at = ((lk + 2) * kMidS + lj + 2) * nh + I;
        const uint32_t q = prow(Lf, j0 + lj, k0 + lk) + (uint32_t)I;
        se += E0[at];
        if (want_x) sx = p.add_x(q, 0, sx);
        sd += Z[(lk * kMidT + lj) * nh + I];
        if (both) sd += Z[own_cells + (lk * kMidT + lj) * nh + I];
        se += E1[at];
        if (want_x) sx = p.add_x(half + q, 1, sx);
      }
    const uint32_t pc = pk_of(Lc, I, j0 / 2 + cj, k0 / 2 + ck);
    if constexpr (P::kShift) {
      store_coarse_corr(pc, se, sd, sx, eH, nullptr, rhoH, XH, Xf, rx);
    } else {
      rhoH[pc] = sd * 0.125f;
      if (eH) eH[pc] = 0.0f;
    }
  }
}

// The way up: e += P c on colour 1 (old values in ea), then both half-sweeps;
// writes both colours of e.
template <class P>
__device__ __forceinline__ void mid_up(const Lev& Lf, const Lev& Lc, const P& p,
                                       const float* __restrict__ ea, const float* __restrict__ c,
                                       float* __restrict__ e, uint32_t tile, float* lds) {
  const int n = Lf.n, nh = Lf.nh, nt = n / kMidT, nc = Lc.n;
  const uint32_t half = (uint32_t)Lf.half;
  const int tk = (int)tile / nt, j0 = ((int)tile - tk * nt) * kMidT, k0 = tk * kMidT;
  float* E0 = lds;
  float* E1 = E0 + kMidS * kMidS * nh;
  float* W = E1 + kMidS * kMidS * nh;  // coarse rows J0-2 .., K0-2 .., natural order
  const int J0 = j0 / 2 - 2, K0 = k0 / 2 - 2;
  for (int g = threadIdx.x; g < kMidSC * kMidSC * nc; g += kMidThreads) {
    const int row = (int)Lf.dnh.div((uint32_t)g), I = g - row * nc;
    int J = J0 + row % kMidSC, K = K0 + row / kMidSC;
    J = J < 0 ? J + nc : (J >= nc ? J - nc : J);
    K = K < 0 ? K + nc : (K >= nc ? K - nc : K);
    W[g] = c[pk_of(Lc, I, J, K)];
  }
  __syncthreads();
  const int all = kMidS * kMidS * nh;
  for (int g = threadIdx.x; g < all; g += kMidThreads) {
    const int row = (int)Lf.dnh.div((uint32_t)g), ih = g - row * nh;
    const MidRow r = mid_row(row, j0, k0, n);
    if (r.dist > 2) continue;
    // frame row rj is fine row j0 - 2 + rj (j0 even): coarse row rj/2 + 1 of W
    const int Jn = r.rj / 2 + 1, Jf = (r.rj & 1) ? Jn + 1 : Jn - 1;
    const int Kn = r.rk / 2 + 1, Kf = (r.rk & 1) ? Kn + 1 : Kn - 1;
    const int x = (1 + r.j + r.k) & 1;
    const int Ifar = x ? (ih + 1 == nc ? 0 : ih + 1) : (ih == 0 ? nc - 1 : ih - 1);
    auto ax = [&](int J, int K) {
      const float* w = W + (K * kMidSC + J) * nc;
      return p34<float>(w[ih], w[Ifar]);
    };
    const float ayn = p34<float>(ax(Jn, Kn), ax(Jf, Kn));
    const float ayf = p34<float>(ax(Jn, Kf), ax(Jf, Kf));
    E1[g] = ea[prow(Lf, r.j, r.k) + (uint32_t)ih] + p34<float>(ayn, ayf);
  }
  __syncthreads();
  for (int g = threadIdx.x; g < all; g += kMidThreads) {
    const int row = (int)Lf.dnh.div((uint32_t)g), ih = g - row * nh;
    const MidRow r = mid_row(row, j0, k0, n);
    if (r.dist > 1) continue;
    const uint32_t q = prow(Lf, r.j, r.k) + (uint32_t)ih;
    const float v = p.update(p.load(q), mid_sum(E1, row, ih, nh, (r.j + r.k) & 1));
    E0[g] = v;
    if (r.dist == 0) e[q] = v;
  }
  __syncthreads();
  for (int g = threadIdx.x; g < kMidT * kMidT * nh; g += kMidThreads) {
    const int own = (int)Lf.dnh.div((uint32_t)g), ih = g - own * nh;
    const int j = j0 + own % kMidT, k = k0 + own / kMidT;
    const int row = (own / kMidT + 2) * kMidS + own % kMidT + 2;
    const uint32_t q = half + prow(Lf, j, k) + (uint32_t)ih;
    e[q] = p.update(p.load(q), mid_sum(E0, row, ih, nh, (j + k + 1) & 1));
  }
}

template <class P>
__global__ __launch_bounds__(kMidThreads) void k_mid_down(Lev Lf, Lev Lc, P p, const float* e,
                                                          float* ea, float* eH, float* rhoH,
                                                          float* XH, float* Xf, int rx, int fresh) {
  extern __shared__ __align__(16) unsigned char mid_lds[];
  mid_down(Lf, Lc, p, e, ea, eH, rhoH, XH, Xf, rx, fresh, blockIdx.x,
           reinterpret_cast<float*>(mid_lds));
}
template <class P>
__global__ __launch_bounds__(kMidThreads) void k_mid_up(Lev Lf, Lev Lc, P p, const float* ea,
                                                        const float* c, float* e) {
  extern __shared__ __align__(16) unsigned char mid_lds[];
  mid_up(Lf, Lc, p, ea, c, e, blockIdx.x, reinterpret_cast<float*>(mid_lds));
}

}  // namespace mgg
