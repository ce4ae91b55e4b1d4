// Kernel templates of the bandwidth-optimised regression (Sec. 3), instantiated
// per feature count beside the regression kernels.  The estimator and its
// launcher are described in esim_bandwidth.hip.
//
// A candidate h only changes the weights: with the plan's regressors v the
// exponent is multiplied by (h / h_k)^2, the unknowns and the ridge stay those of
// the plan's units.  So every candidate runs the regression's window walk (dense
// tiles from LDS, work lists 16 lanes per item) with a scaled exponent, and its
// system is the regression's; v = A^-1 e_0 is a second solve on the factor.  Bound
// by VALU issue: five candidates at every pixel of a 480 x 360 frame (F = 7,
// r = 7, three frames) take 1.70 ms, 2.87 ms when every candidate read its
// windows column by column from memory.
#pragma once

#include "esim_bandwidth.h"
#include "esim_regress_impl.h"

namespace esim {
namespace {

// Solves candidate k of item idx (pixel pix) from its window sums and writes its
// outputs if its SURE beats the best so far (NaN, a failed factor, never does).
template <int F>
__device__ __forceinline__ void solve_candidate(const BandwidthArgs& b, const ClipDev& C, int k, int64_t idx,
                                                int64_t pix, const Gram<F, double>& gm, double& best) {
  constexpr int P = F + 3;
  const RegressArgs& a = b.reg;
  const int64_t cen = static_cast<int64_t>(a.t) * C.HW + pix;
  double M[P * (P + 1) / 2], th[P], rhs[P], e0[P], v[P], anorm;
  const double iW = gram_solve<F, double>(gm, C, M, rhs, th, anorm);
  (void)anorm;
#pragma unroll
  for (int i = 0; i < P; ++i) e0[i] = i == 0 ? 1.0 : 0.0;
  chol_solve<P, double>(M, e0, v);
  const double s2 = b.vy[cen];
  const double d = th[0] - static_cast<double>(C.y[cen]);
  const double sure = d * d + 2.0 * s2 * v[0] * iW - s2;
  if (k == 0) {                       // what stays if every factor fails
    a.alpha[idx] = __builtin_nanf("");
    if (b.hsel) b.hsel[idx] = __builtin_nanf("");
    if (b.sure) b.sure[idx] = __builtin_nanf("");
  }
  if (sure < best) {
    best = sure;
    a.alpha[idx] = static_cast<float>(th[0]);
    if (a.beta)
#pragma unroll
      for (int i = 0; i < F + 2; ++i) a.beta[i * a.n_out + idx] = static_cast<float>(th[1 + i] * C.sf[i]);
    if (b.hsel) b.hsel[idx] = static_cast<float>(b.h[k]);
    if (b.sure) b.sure[idx] = static_cast<float>(sure);
  }
}

// Dense, windows in LDS: a tile per wave.
template <int F, bool F16>
__global__ void __launch_bounds__(256 * regress_waves_per_simd(F, false))
__attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
bandwidth_tile_kernel(BandwidthArgs b) {
  extern __shared__ float4 tile_lds[];
  __shared__ int taken;
  const RegressArgs& a = b.reg;
  float4* lds = tile_lds + uni(static_cast<int>(threadIdx.x) / kWave) * a.tile_units;
  const GroupQueue queue(a.n_dense_groups, 1, a.nxcd, &taken);
  const ClipDev& C = a.clips[0];
  for (int64_t q = queue.start(); q < queue.count; q = queue.next()) {
    double best = INFINITY;
#pragma unroll 1
    for (int k = 0; k < b.K; ++k) {
      TileGeom<F, F16> geo;
      make_tile(geo, C, static_cast<int>(queue.group(q)), a.t, uni(b.scale[k] * b.scale[k]));
      Gram<F, double> gm;
      tile_gram(geo, lds, gm);
      if (geo.px < geo.W && geo.py < geo.H) {
        const int64_t pix = static_cast<int64_t>(geo.py) * geo.W + geo.px;
        solve_candidate<F>(b, C, k, pix, pix, gm, best);
      }
    }
  }
}

// Dense, windows too wide for LDS: a lane per pixel, from memory.
template <int F, bool F16>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
bandwidth_dense_kernel(BandwidthArgs b) {
  const RegressArgs& a = b.reg;
  const int lane = threadIdx.x & (kWave - 1);
  GroupIter it(a.n_dense_groups, a.nxcd);
  int64_t g;
  while (it.next(g)) {
    int cl, t;
    int64_t pix, idx;
    const bool valid = group_item<1>(a, g, lane, 0, cl, pix, t, idx);
    double best = INFINITY;
#pragma unroll 1
    for (int k = 0; k < b.K; ++k)
      window_grams<F, 1, F16>(a, valid, cl, pix, t, 0,
                                     [&](const ClipDev& C, bool active, int64_t p, int, Gram<F, double>& gm) {
        if (active) solve_candidate<F>(b, C, k, idx, p, gm, best);
      }, uni(b.scale[k] * b.scale[k]));
  }
}

// Work lists and small frames: the list regression's rounds, once per candidate.  An item's best
// SURE stays in LDS and its fields are read again for each solve: held in registers over the
// walks they were spilled there (F = 7, r = 5, one frame, 500 items 46.5 us, now 42.1).
template <int F, bool F16, int KIND>
__global__ void __launch_bounds__(256 * regress_waves_per_simd(F, false))
__attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
bandwidth_list_kernel(BandwidthArgs b) {
  constexpr int L = 16, G = kWave / L;
  using R = ListRound<F, L>;
  __shared__ double parked[R::ITEMS * R::STRIDE];
  __shared__ double best[R::ITEMS];
  __shared__ int taken;
  const RegressArgs& a = b.reg;
  const int64_t n_items =
      a.items ? max(static_cast<int64_t>(0), min(static_cast<int64_t>(a.count[0]), a.n_out)) : 0;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = item_slot<L>(lane), j = item_lane<L>(lane);
  const GroupQueue queue(a.items ? (n_items + G - 1) / G : a.n_dense_groups, 1, a.nxcd, &taken);
  for (int64_t k0 = 0; k0 < queue.count; k0 += R::GROUPS) {
    const int n = static_cast<int>(min(static_cast<int64_t>(R::GROUPS), queue.count - k0));
#pragma unroll 1
    for (int k = 0; k < b.K; ++k) {
      for (int64_t q = queue.start(); q < n; q = queue.next()) {
        int cl, t;
        int64_t pix, idx;
        const bool valid = group_item<L>(a, queue.group(k0 + q), slot, n_items, cl, pix, t, idx);
        double* to = parked + (static_cast<int>(q) * G + slot) * R::STRIDE + j;
        park_group<F, L, F16, KIND>(a, valid, cl, pix, t, j, to, uni(b.scale[k] * b.scale[k]));
      }
      __syncthreads();
      if (threadIdx.x == 0) *queue.taken = static_cast<int>(blockDim.x / kWave);
      const int i = threadIdx.x;                // the item of the round that this thread solves
      int cl, t;
      int64_t pix, idx;
      if (i < n * G && group_item<L>(a, queue.group(k0 + i / G), i % G, n_items, cl, pix, t, idx)) {
        double least = k == 0 ? INFINITY : best[i];
        Gram<F, double> gm;
        parked_gram<F, L>(parked + i * R::STRIDE, gm);
        solve_candidate<F>(b, a.clips[0], k, idx, pix, gm, least);
        best[i] = least;
      }
      __syncthreads();
    }
  }
}

}  // namespace
}  // namespace esim
