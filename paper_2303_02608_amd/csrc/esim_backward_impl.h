// Item kernel of the adjoint (esim_backward.hip), instantiated per feature count
// beside the regression kernels: the list regression's window sums (groups from
// the block's queue, totals parked in LDS, one lane per item factors and solves),
// then theta, v = A^-1 e_0 and the item's record.  Bound like the list regression by VALU issue
// and the window loads.
#pragma once

#include "esim_backward.h"
#include "esim_regress_impl.h"

namespace esim {
namespace {

template <int F, int L, bool F16, int KIND>
__global__ void __launch_bounds__(256 * regress_waves_per_simd(F, false))
__attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
adjoint_kernel(AdjointArgs b) {
  constexpr int P = F + 3;
  constexpr int REC = adjoint_record(F);
  constexpr int G = kWave / L;
  using R = ListRound<F, L>;
  __shared__ double parked[R::ITEMS * R::STRIDE];
  __shared__ int taken;
  const RegressArgs& a = b.reg;
  const int64_t n_items = b.bd.n;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = item_slot<L>(lane), j = item_lane<L>(lane);
  const GroupQueue queue((n_items + G - 1) / G, 1, a.nxcd, &taken);
  int64_t k = queue.start();
  for (int64_t k0 = 0; k0 < queue.count; k0 += R::GROUPS) {
    const int64_t end = min(k0 + R::GROUPS, queue.count);
    for (; k < end; k = queue.next()) {
      int cl, t;
      int64_t pix, idx;
      const bool valid = group_item<L>(a, queue.group(k), slot, n_items, cl, pix, t, idx) && b.g_alpha[idx] != 0.0f;
      double* to = parked + (static_cast<int>(k - k0) * G + slot) * R::STRIDE + j;
      park_group<F, L, F16, KIND>(a, valid, cl, pix, t, j, to);
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (i < static_cast<int>(end - k0) * G) {
      int cl, t;
      int64_t pix, idx;
      if (group_item<L>(a, queue.group(k0 + i / G), i % G, n_items, cl, pix, t, idx)) {
        const float g = b.g_alpha[idx];
        if (g != 0.0f) {
          const ClipDev& C = a.clips[0];
          Gram<F, double> gm;
          parked_gram<F, L>(parked + i * R::STRIDE, gm);
          double M[P * (P + 1) / 2], rhs[P], th[P], e0[P], vv[P], anorm;
          const double iW = gram_solve<F, double>(gm, C, M, rhs, th, anorm);
          (void)anorm;
#pragma unroll
          for (int u = 0; u < P; ++u) e0[u] = u == 0 ? 1.0 : 0.0;
          chol_solve<P, double>(M, e0, vv);
          double vLt = 0.0;      // v^T Lambda theta (Lambda = scaled ridge on the beta block)
#pragma unroll
          for (int u = 1; u < P; ++u) vLt = fma(vv[u] * (C.ridge * C.c2[u - 1]), th[u], vLt);
          const double gw = static_cast<double>(g) * iW;
          double* o = b.bd.rec + idx * REC;
#pragma unroll
          for (int u = 0; u < P; ++u) {
            o[u] = gw * vv[u];
            o[P + u] = th[u];
          }
          o[2 * P] = gw * vLt;
#pragma unroll
          for (int f = 0; f < F; ++f)
            o[2 * P + 1 + f] = static_cast<double>(feat_value(C, t, f, pix)) * C.sf[2 + f];
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace
}  // namespace esim
