// Weighted local regression (Sec. 2.1, eqs. 3-5) on gfx950: kernel templates.
// Each feature count is instantiated in a translation unit of its own
// (esim_regress_inst.hip); esim_regress.hip dispatches.
//
// One regression ("item") is the minimiser of
//     (1/W) sum_i w_i (y_i - alpha - beta^T u_i)^2 + ridge * |beta|^2,
//     u_i = x^i - x^c,  w_i = exp(-1/2 sum_j (u_ij / (h b_j))^2),  W = sum_i w_i,
// over the window |dx|, |dy| <= r, |dt| <= tr (truncated at image borders and
// clip ends), with x = (px / r, py / r, f_0 .. f_{F-1}).
//
// Mapping.  Dense launches: one lane per pixel and a tile of 64 pixels per wave,
// its window rows in LDS (regress_tile_kernel).  Work lists: 16 lanes per item,
// one window column each, 4 items per wave (regress_list_kernel; 4 and 8 lanes
// are compiled too), and small dense frames.  Instances of 1 and 2 lanes per item
// (regress_kernel) read their windows from memory: dense windows too wide for LDS,
// images narrower than half a tile, and the condition output.  Which one a clip
// takes follows from the clip alone (esim_schedule.h).  In all of them a coordinate is constant over a line of samples and the
// other over a cell, and no entry with a coordinate factor is summed per sample
// (esim_wlr.h): 87 VALU instructions per sample at F = 7 and three frames.
//
// What bounds them: VALU issue.  With every CU busy the clock falls to 2.0 GHz
// (2.5 GHz with 16 CUs busy); at that clock a dense launch of many tiles issues
// a VALU instruction in each of its SIMDs' slots (2048 x 256 pixels, r = 7, three
// frames: 0.94 ms; one lane per pixel from memory took 1.30 ms).  A list of
// 18 400 items takes 60 us (75 us with the solve in every lane and one row of
// loads ahead), of which about 15 us are the launch, the first loads and the
// last solve.
//
// Precision.  The weight exponent is summed in FP64 from FP64 differences of
// the FP32 inputs and exponentiated with the FP32 hardware exp2 (about 1e-7
// relative).  Gram, right-hand side and Cholesky are FP64: without packed FP32
// (disabled by the compile flags) an FP64 FMA issues at the same rate as an
// FP32 one on CDNA4, and the windows are ill-conditioned (kappa up to ~1e6
// with a 1e-6 ridge), which FP32 accumulation does not survive at the 1e-4
// contract.
//
// The lane partials of an item are then summed so that each total ends in one
// lane (scatter_sum), parked in LDS, and solved by one lane per item in registers
// (1 and 2 lanes per item: summed in every lane and solved there).  The optional
// condition output is Hager's 1-norm estimate on the factor.
#pragma once
#include <type_traits>

#include "esim_wlr.h"

namespace esim {
namespace {

// Item i of a work list, checked (clip, pixel, frame); false for padding and
// entries outside the plan.
__device__ __forceinline__ bool list_item(const RegressArgs& a, int64_t i, int64_t n_items, int& cl, int64_t& pix,
                                          int& t) {
  const int64_t it = i < n_items ? a.items[i] : -1;
  if (it < 0) return false;
  const int c = item_clip(it);
  if (c >= a.nclips) return false;
  const int64_t p = item_pixel(it);
  const int fr = a.t >= 0 ? a.t : item_frame(it);
  if (p >= a.clips[c].HW || fr < 0 || fr >= a.clips[c].T) return false;
  cl = c;
  pix = p;
  t = fr;
  return true;
}

// Item `slot` of group g (G items per group): work-list entry g * G + slot, or
// pixel slot of the group's G pixels (dense).  idx is its output index.
template <int L>
__device__ __forceinline__ bool group_item(const RegressArgs& a, int64_t g, int slot, int64_t n_items, int& cl,
                                           int64_t& pix, int& t, int64_t& idx) {
  constexpr int G = kWave / L;
  cl = 0;
  pix = 0;
  t = a.t;
  if (a.items) {
    idx = g * G + slot;
    return list_item(a, idx, n_items, cl, pix, t);
  }
  for (int c = 1; c < a.nclips; ++c)
    if (a.clips[c].first_group <= g) cl = c;
  const int64_t p = (g - a.clips[cl].first_group) * G + slot;
  const bool valid = p < a.clips[cl].HW && a.t < a.clips[cl].T;
  pix = valid ? p : 0;
  idx = a.clips[cl].pix_off + p;
  return valid;
}

// Residual of eq. (4) at the solution: (A + Lambda) theta = rhs, so
// R = Syy/W - theta^T rhs - theta^T Lambda theta.
template <int F>
__device__ __forceinline__ double residual(const ClipDev& C, const double (&th)[F + 3], const double (&rhs)[F + 3],
                                           double syy_w) {
  double tg = 0.0, bb = 0.0;
#pragma unroll
  for (int i = 0; i < F + 3; ++i) tg = fma(th[i], rhs[i], tg);
#pragma unroll
  for (int i = 1; i < F + 3; ++i) bb = fma(th[i] * C.c2[i - 1], th[i], bb);
  return syy_w - tg - C.ridge * bb;
}

// Writes item idx (pixel pix of clip C at frame t).  The L lanes of an item
// share the writes: lane j writes components j, j + L, ...; each component's
// value is picked by a select over the L candidates of its round, so a lane
// forms one address per round instead of one per component.
template <int F, int L>
__device__ __forceinline__ void write_item(const RegressArgs& a, const ClipDev& C, int64_t idx, int64_t pix, int t,
                                           int j, const double (&th)[F + 3], const double (&rhs)[F + 3],
                                           double syy_w, bool has_kappa, double kap) {
  constexpr int D = F + 2;
  if (a.update_state) {
    if (j == 0) {
      C.st_alpha[pix] = static_cast<float>(th[0]);
      C.st_tref[pix] = t;
    }
#pragma unroll
    for (int k = 0; k < (F + L - 1) / L; ++k) {
      const int f = j + k * L;
      if (f < F) {
        double bv = 0.0;
#pragma unroll
        for (int ff = k * L; ff < (k + 1) * L && ff < F; ++ff)
          if (ff == f) bv = th[3 + ff] * C.sf[2 + ff];
        C.st_beta[f * C.HW + pix] = static_cast<float>(bv);
        C.st_xref[f * C.HW + pix] = feat_value(C, t, f, pix);
      }
    }
  }
  if (a.alpha) {
    if (j == 0) {
      a.alpha[idx] = static_cast<float>(th[0]);
      if (a.resid) a.resid[idx] = static_cast<float>(residual<F>(C, th, rhs, syy_w));
      if (a.kappa && has_kappa) a.kappa[idx] = static_cast<float>(kap);
    }
    if (a.beta) {
#pragma unroll
      for (int k = 0; k < (D + L - 1) / L; ++k) {
        const int d = j + k * L;
        if (d < D) {
          double bv = 0.0;
#pragma unroll
          for (int dd = k * L; dd < (k + 1) * L && dd < D; ++dd)
            if (dd == d) bv = th[1 + dd] * C.sf[dd];
          a.beta[static_cast<int64_t>(d) * a.n_out + idx] = static_cast<float>(bv);
        }
      }
    }
  }
}

// The items of one wave's group: calls fn(C, geo, active, pix, t) for the lanes'
// items with their walk's geometry (weights to the power wscale).  Rounds over the
// (clip, first frame, frame count) present in the wave, so that those are uniform
// in the walk: nearly always one round.
template <int F, bool F16, class Fn>
__device__ __forceinline__ void group_rounds(const RegressArgs& a, bool valid, int my_cl, int64_t my_pix, int my_t,
                                             double wscale, Fn&& fn) {
  uint64_t todo = __ballot(valid);
  while (todo != 0) {
    const int src = __ffsll(static_cast<unsigned long long>(todo)) - 1;
    const int cl = __builtin_amdgcn_readlane(my_cl, src);
    const int t0 = __builtin_amdgcn_readlane(my_t, src);
    const int p0 = __builtin_amdgcn_readlane(static_cast<int>(my_pix), src);
    const ClipDev& C = a.clips[cl];
    const int tr = uni(C.tr), T = uni(C.T);
    const int lo = max(-tr, -t0), hi = min(tr, T - 1 - t0);
    const bool active = valid && my_cl == cl && max(-tr, -my_t) == lo && min(tr, T - 1 - my_t) == hi;
    todo &= ~__ballot(active);
    // lanes of other rounds (or without an item) walk the first item's window
    // with weight 0
    const int64_t pix = active ? my_pix : static_cast<int64_t>(p0);
    const int t = active ? my_t : t0;
    // frames held by the buffer resources: the window of a uniform frame, or
    // the whole clip when items carry their own frame
    const int f0 = a.t >= 0 ? max(0, a.t - tr) : 0;
    const int f1 = a.t >= 0 ? min(T, a.t + tr + 1) : T;
    WalkGeom<F, F16> geo;
    make_walk(geo, C, pix, t, lo, hi - lo + 1, f0, f1, active, wscale);
    fn(C, geo, active, pix, t);
  }
}

// The same with the window sums `got` of the lane's part of its item (the columns
// j, j + L, ...): fn(C, active, pix, t, got).
template <int F, int L, bool F16, class Fn>
__device__ __forceinline__ void window_grams(const RegressArgs& a, bool valid, int my_cl, int64_t my_pix, int my_t,
                                             int j, Fn&& fn, double wscale = 1.0) {
  group_rounds<F, F16>(a, valid, my_cl, my_pix, my_t, wscale,
                       [&](const ClipDev& C, const WalkGeom<F, F16>& geo, bool active, int64_t pix, int t) {
    Gram<F, double> got;
    walk_gram<F, L, F16>(geo, j, a.items == nullptr, got);
    fn(C, active, pix, t, got);
  });
}

// The groups of one wave of an instance of 1 or 2 lanes per item, FP64 Gram: every
// lane of an item factors and solves.  KAPPA: the instance that writes the
// condition estimate (one lane per item); the estimate's code stays out of the
// other instances, whose register budget it would raise.
template <int F, int L, bool F16, bool KAPPA>
__device__ __forceinline__ void regress_groups(const RegressArgs& a, GroupIter& it, int64_t n_items) {
  constexpr int P = F + 3;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = lane / L, j = lane % L;
  int64_t g;
  while (it.next(g)) {
    int cl, t;
    int64_t pix, idx;
    const bool valid = group_item<L>(a, g, slot, n_items, cl, pix, t, idx);
    window_grams<F, L, F16>(a, valid, cl, pix, t, j,
                            [&](const ClipDev& C, bool active, int64_t ipix, int it_t, Gram<F, double>& gm) {
      gm.template lane_sum<L>();
      double M[P * (P + 1) / 2], th[P], rhs[P], anorm, kap = 0.0;
      const double iW = gram_solve<F, double>(gm, C, M, rhs, th, anorm);
      const double syy_w = gm.Syy * iW;
      if constexpr (KAPPA) {
        equilibrate_factor<P, double>(M);
        kap = anorm * hager_inv_norm1<P, double>(M);
      } else {
        (void)anorm;
      }
      if (active) write_item<F, L>(a, C, idx, ipix, it_t, j, th, rhs, syy_w, KAPPA, kap);
    });
  }
}

// Instances of 4, 8 or 16 lanes per item (work lists; small dense frames): one
// block per CU takes a run of groups, a round of up to kRoundItems items at a
// time.  A wave leaves the totals of its groups' items in the block's LDS; when
// the round's groups are done, one lane per item factors, solves and writes.
// Solving in every lane of an item right after its walk took 1400 of a 4-item
// group's 6200 VALU instructions at F = 7 (16 lanes): here the lane sums take 250
// and the solve is shared by the round.
template <int F, int L>
struct ListRound {
  static constexpr int WAVES = 4 * regress_waves_per_simd(F, false);
  static constexpr int ITEMS = 16 * WAVES;                          // of a round
  static constexpr int GROUPS = ITEMS * L / kWave;
  static constexpr int NE = (F + 4) * (F + 5) / 2;                  // totals of an item
  static constexpr int REGS = (NE + L - 1) / L;
  static constexpr int STRIDE = REGS * L + 1;                       // odd: neighbouring items on other banks
};

// Walks the items of a group and parks their totals: lane j's share of item
// `slot` goes to to[q L], to being the lane's place in the item's parking space.
template <int F, int L, bool F16, int KIND>
__device__ __forceinline__ void park_group(const RegressArgs& a, bool valid, int cl, int64_t pix, int t, int j,
                                           double* to, double wscale = 1.0) {
  using R = ListRound<F, L>;
  const int lane = threadIdx.x & (kWave - 1);
  group_rounds<F, F16>(a, valid, cl, pix, t, wscale,
                       [&](const ClipDev&, const WalkGeom<F, F16>& geo, bool active, int64_t, int) {
    auto park = [&](Gram<F, double>& got, bool first) {
      double s[R::NE];
      int e = 0;
      got.each([&](double& v) { s[e++] = v; });
      scatter_sum<L>(s, lane);
      if (active) {
#pragma unroll
        for (int q = 0; q < R::REGS; ++q) to[q * L] = first ? s[q] : to[q * L] + s[q];
      }
    };
    if constexpr (L == 4 && F <= 4) {
      // few sums, and many turns to add them over the lanes in: kept in registers
      // over the turns (F = 3, r = 3, 20000 items 14.1 -> 12.3 us; F = 10 694 -> 699)
      Gram<F, double> got;
      walk_gram<F, L, F16>(geo, j, true, got);
      park(got, true);
    } else {
      walk_parts<F, L, F16, KIND>(geo, j, park);
    }
  });
}

// The totals of a parked item.
template <int F, int L>
__device__ __forceinline__ void parked_gram(const double* at, Gram<F, double>& gm) {
  int e = 0;
  gm.each([&](double& v) { v = at[total_pos<L>(e++)]; });
}

template <int F, int L, bool F16, int KIND>
__global__ void __launch_bounds__(256 * regress_waves_per_simd(F, false))
__attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
regress_list_kernel(RegressArgs a) {
  using R = ListRound<F, L>;
  constexpr int G = kWave / L;
  constexpr int P = F + 3;
  __shared__ double parked[R::ITEMS * R::STRIDE];
  const int64_t n_items =
      a.items ? max(static_cast<int64_t>(0), min(static_cast<int64_t>(a.count[0]), a.n_out)) : 0;
  const int64_t ngroups = a.items ? (n_items + G - 1) / G : a.n_dense_groups;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = item_slot<L>(lane), j = item_lane<L>(lane);
  __shared__ int taken;
  const GroupQueue queue(ngroups, a.nclips, a.nxcd, &taken);
  int64_t k = queue.start();
  for (int64_t k0 = 0; k0 < queue.count; k0 += R::GROUPS) {
    const int64_t end = min(k0 + R::GROUPS, queue.count);
    const int n = static_cast<int>(end - k0);
    // a wave keeps a group that it fetched beyond the round for the next one
    for (; k < end; k = queue.next()) {
      int cl, t;
      int64_t pix, idx;
      const bool valid = group_item<L>(a, queue.group(k), slot, n_items, cl, pix, t, idx);
      double* to = parked + (static_cast<int>(k - k0) * G + slot) * R::STRIDE + j;
      park_group<F, L, F16, KIND>(a, valid, cl, pix, t, j, to);
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (i < n * G) {
      int cl, t;
      int64_t pix, idx;
      if (group_item<L>(a, queue.group(k0 + i / G), i % G, n_items, cl, pix, t, idx)) {
        const ClipDev& C = a.clips[cl];
        Gram<F, double> gm;
        parked_gram<F, L>(parked + i * R::STRIDE, gm);
        double M[P * (P + 1) / 2], th[P], rhs[P], anorm;
        const double iW = gram_solve<F, double>(gm, C, M, rhs, th, anorm);
        (void)anorm;
        write_item<F, 1>(a, C, idx, pix, t, 0, th, rhs, gm.Syy * iW, false, 0.0);
      }
    }
    __syncthreads();
  }
}

// The groups of one wave, reduced precision: FP32 regressors and weights, FP32
// Gram with block-compensated sums (GramC), FP32 Cholesky, and an FP64 re-solve
// of the same compensated Gram for items whose Hager condition estimate exceeds
// kappa_fp64.
template <int F, int L, bool F16>
__device__ __forceinline__ void regress_groups_c32(const RegressArgs& a, GroupIter& it, int64_t n_items) {
  constexpr int P = F + 3;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = lane / L, j = lane % L;
  int64_t g;
  while (it.next(g)) {
    int my_cl, my_t;
    int64_t my_pix, idx;
    const bool valid = group_item<L>(a, g, slot, n_items, my_cl, my_pix, my_t, idx);
    // rounds over the clips present in the wave
    uint64_t todo = __ballot(valid);
    while (todo != 0) {
      const int cl = __builtin_amdgcn_readlane(my_cl, __ffsll(static_cast<unsigned long long>(todo)) - 1);
      const bool active = valid && my_cl == cl;
      todo &= ~__ballot(active);
      const ClipDev& C = a.clips[cl];
      const int f0 = a.t >= 0 ? max(0, a.t - C.tr) : 0;
      const int f1 = a.t >= 0 ? min(C.T, a.t + C.tr + 1) : C.T;
      ItemGeom<F, F16, float> geo;
      make_geom(geo, C, active ? my_pix : 0, active ? my_t : (a.t >= 0 ? a.t : 0), f0, f1, active);
      double th[P], rhs[P];
      GramC<F> gc;
      gc.zero();
      window_loop<F, L, F16, float>(
          geo, j, [&](float) { gc.pass_begin(); },
          [&](float w, float yd, const float (&v)[F], float vy, int, int, int, bool) { gc.add(w, yd, v, vy); },
          [&](float vx) { gc.pass_end(vx); });
      gc.template lane_sum<L>();
      Gram<F, float> g32;
      gc.values(g32);
      float M32[P * (P + 1) / 2], r32[P], t32[P], an32;
      double iW = gram_solve<F, float>(g32, C, M32, r32, t32, an32);
      equilibrate_factor<P, float>(M32);
      const double kap = static_cast<double>(an32) * static_cast<double>(hager_inv_norm1<P, float>(M32));
      const bool fallback = !(kap <= C.kappa_fp64);
      double Syy = g32.Syy;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        th[i] = t32[i];
        rhs[i] = r32[i];
      }
      if (__ballot(fallback && active) != 0) {
        Gram<F, double> g64;
        gc.values(g64);
        double M[P * (P + 1) / 2], r64[P], t64[P], an64;
        const double iW64 = gram_solve<F, double>(g64, C, M, r64, t64, an64);
        if (fallback) {
          iW = iW64;
          Syy = g64.Syy;
#pragma unroll
          for (int i = 0; i < P; ++i) {
            th[i] = t64[i];
            rhs[i] = r64[i];
          }
        }
      }
      if (active) write_item<F, L>(a, C, idx, my_pix, my_t, j, th, rhs, Syy * iW, true, kap);
    }
  }
}

// Dense launches with one lane per pixel whose windows fit LDS: a tile per wave
// (tile_frames), one block per CU.
template <int F, bool F16>
__global__ void __launch_bounds__(256 * regress_waves_per_simd(F, false))
__attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, false))))
regress_tile_kernel(RegressArgs a) {
  constexpr int P = F + 3;
  extern __shared__ float4 tile_lds[];
  __shared__ int taken;
  float4* lds = tile_lds + uni(static_cast<int>(threadIdx.x) / kWave) * a.tile_units;
  const GroupQueue queue(a.n_dense_groups, a.nclips, a.nxcd, &taken);
  for (int64_t k = queue.start(); k < queue.count; k = queue.next()) {
    const int64_t g = queue.group(k);
    int cl = 0;
    for (int c = 1; c < a.nclips; ++c)
      if (a.clips[c].first_group <= g) cl = c;
    const ClipDev& C = a.clips[cl];
    if (a.t >= C.T) continue;
    TileGeom<F, F16> geo;
    make_tile(geo, C, static_cast<int>(g - C.first_group), a.t);
    Gram<F, double> gm;
    tile_gram(geo, lds, gm);
    double M[P * (P + 1) / 2], th[P], rhs[P], anorm;
    const double iW = gram_solve<F, double>(gm, C, M, rhs, th, anorm);
    (void)anorm;
    if (geo.px < geo.W && geo.py < geo.H) {
      const int64_t pix = static_cast<int64_t>(geo.py) * geo.W + geo.px;
      write_item<F, 1>(a, C, C.pix_off + pix, pix, a.t, 0, th, rhs, gm.Syy * iW, false, 0.0);
    }
  }
}

template <int F, int L, bool F16, bool C32, bool KAPPA = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(regress_waves_per_simd(F, C32))))
regress_kernel(RegressArgs a) {
  constexpr int G = kWave / L;
  // the device count is clamped to the output length: item i writes index i
  const int64_t n_items =
      a.items ? max(static_cast<int64_t>(0), min(static_cast<int64_t>(a.count[0]), a.n_out)) : 0;
  const int64_t ngroups = a.items ? (n_items + G - 1) / G : a.n_dense_groups;
  GroupIter it(ngroups, a.nxcd, a.items ? nullptr : a.xcd_bounds);
  if constexpr (C32) regress_groups_c32<F, L, F16>(a, it, n_items);
  else regress_groups<F, L, F16, KAPPA>(a, it, n_items);
}

}  // namespace
}  // namespace esim
