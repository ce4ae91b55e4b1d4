// Adjoint of the regression estimate alpha (Sec. 2.1, eqs. 4-5 differentiated).
//
// With A the W-normalised Gram plus ridge Lambda (in bandwidth-scaled units),
// theta = A^{-1} g, v = A^{-1} e_0, s_i = v^T z_i and r_i = y_i - z_i^T theta:
//     d alpha / d y_i = (w_i / W) s_i
//     d alpha / d w_i = (s_i r_i - v^T Lambda theta) / W
//     d w_i / d b_j   = w_i u_ij^2 / (h^2 b_j^3) = w_i v_ij^2 / b_j
// (alpha does not depend on the scaling of the regressors, so the scaled system
// gives the same derivatives).
//
// Kernels, all deterministic (no atomics on values):
//   fill_map / map_items  a dense (frame, pixel) -> item index map
//   adjoint_kernel        (esim_backward_impl.h) per item: the window's Gram,
//                         Cholesky, theta and v (the window is recomputed, not
//                         stored by the forward pass); writes the item's record c = g_alpha v / W,
//                         theta, q = g_alpha v^T Lambda theta / W
//   gather_kernel         per input sample (frame, pixel): for every item whose
//                         window holds it, in a fixed order, recomputes the
//                         sample's weight and regressors from the item's
//                         record, adds w_i c^T z_i to g_y and accumulates
//                         w_i (c^T z_i r_i - q) z_ij^2 for the bandwidths.  A wave
//                         owns 8 x 8 samples and visits the items one at a time,
//                         the record in scalar registers; per-block partials
//   reduce_gb_*           fixed-order two-level sum of the per-block partials
#include "esim_backward.h"
#include "esim_wlr.h"

namespace esim {
namespace {

constexpr int kRedBlocks = 256;
constexpr int kGatherTile = 16;     // input pixels of a gather block: 16 x 16, four waves of 8 x 8
constexpr int kGatherThreads = 256;
constexpr int kGatherWaves = kGatherThreads / kWave;
constexpr int kGatherSlots = 4;              // region slots per thread and step of the gather's scan
constexpr int kGatherCap = kGatherSlots * kGatherThreads;   // listed items: a step's at least

__global__ void __launch_bounds__(256) fill_map_kernel(int32_t* m, int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) m[i] = -1;
}

__device__ __forceinline__ bool item_ok(const ClipDev& C, int64_t it, const float* g_alpha, int64_t i,
                                        int64_t& pix, int& t) {
  if (it < 0 || item_clip(it) != 0) return false;
  pix = item_pixel(it);
  t = item_frame(it);
  return pix < C.HW && t >= 0 && t < C.T && g_alpha[i] != 0.0f;
}

__global__ void __launch_bounds__(256)
map_items_kernel(const ClipDev* __restrict__ clips, const int64_t* __restrict__ items, int64_t n,
                 const float* __restrict__ g_alpha, int32_t* item_map) {
  const ClipDev& C = clips[0];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    int64_t pix;
    int t;
    if (item_ok(C, items[i], g_alpha, i, pix, t)) item_map[static_cast<int64_t>(t) * C.HW + pix] = static_cast<int32_t>(i);
  }
}

// One block per (input frame tq, 16 x 16 tile of input pixels); wave w owns the
// 8 x 8 sub-tile (w & 1, w >> 1), lane l the sample (l & 7, l >> 3) in it.
// The block's item region is the (frame, row, column) slots whose window can
// reach the tile: rows yc, frames tc and columns x within r (tr) of it, taken
// in a fixed order (tc ascending, then yc, then x), 1024 slots per step, four
// per thread.  A step's present items (the frame-pixel map holds their index) are
// listed in that order in LDS (index and position): a wave ballot and prefix per
// set of 256 slots, and the waves' counts exchanged through LDS.  When the list
// would overflow, every wave walks it in order, skipping the items out of reach
// of all of its lanes (64 positions tested per ballot), and each lane whose window
// holds the item adds its sample's terms.  The order of every sum is fixed, so g_y
// and the partials do not depend on scheduling.
//
// The item of a visit is the same for the whole wave, so its record comes through
// scalar loads into SGPRs, one operand of each FMA.  (Staged in LDS, a visit read
// 28 doubles with every lane at one address: 512 bytes a read, 450 cycles of the
// CU's LDS for the four SIMDs against about 55 VALU instructions each.)
template <int F>
__global__ void __launch_bounds__(kGatherThreads) __attribute__((amdgpu_waves_per_eu(F <= 7 ? 5 : 4)))
gather_kernel(const ClipDev* __restrict__ clips, BwdDev bd, float* __restrict__ g_y) {
  constexpr int D = F + 2;
  constexpr int P = F + 3;
  constexpr int R = adjoint_record(F);
  constexpr double K = kHalfLog2e;
  constexpr int cap = kGatherCap;
  using ScalarDouble = const __attribute__((address_space(4))) double;
  __shared__ int2 list[kGatherCap];                             // item, (row << 8) | column
  __shared__ int32_t wcnt[2 * kGatherSlots * kGatherWaves];     // present items per wave and step
  __shared__ double part[kGatherWaves * D];
  const ClipDev& C = clips[0];
  const int r = C.r, tr = C.tr, W = C.W, H = C.H, T = C.T;
  const int ncol = kGatherTile + 2 * r;                        // at most 66 (r <= 25)
  const int ntx = (W + kGatherTile - 1) / kGatherTile;
  const int nty = (H + kGatherTile - 1) / kGatherTile;
  int64_t b = blockIdx.x;
  const int tx = static_cast<int>(b % ntx);
  b /= ntx;
  const int ty = static_cast<int>(b % nty);
  const int tq = static_cast<int>(b / nty);
  const int bx0 = tx * kGatherTile, by0 = ty * kGatherTile;
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  const int wv = static_cast<int>(threadIdx.x) / kWave;
  const int wx0 = bx0 + 8 * (wv & 1), wy0 = by0 + 8 * (wv >> 1);
  const int xq = wx0 + (lane & 7), yq = wy0 + (lane >> 3);
  const bool in = xq < W && yq < H;
  const int xs = bx0 - r;                      // image column of region column 0
  // region columns whose items reach the wave's columns: wc0 .. wc0 + 7 + 2r
  const int wc0 = wx0 - r - xs;
  const int64_t pq = in ? static_cast<int64_t>(yq) * W + xq : 0;
  double fi[F];                                // scaled features
#pragma unroll
  for (int f = 0; f < F; ++f) fi[f] = in ? static_cast<double>(feat_value(C, tq, f, pq)) * C.sf[2 + f] : 0.0;
  const double yi = in ? static_cast<double>(C.y[static_cast<int64_t>(tq) * C.HW + pq]) : 0.0;
  const double vx_step = C.sf[0] / r, vy_step = C.sf[1] / r;
  double acc = 0.0;
  double gb[D];
#pragma unroll
  for (int d = 0; d < D; ++d) gb[d] = 0.0;
  const int t0 = max(0, tq - tr), t1 = min(T - 1, tq + tr);
  const int ntc = t1 - t0 + 1;
  const int yc0 = max(0, by0 - r), yc1 = min(H - 1, by0 + kGatherTile - 1 + r);
  const int nry = yc1 - yc0 + 1;
  // slot s: row k = s / ncol = (tc - t0) nry + yc - yc0, column s % ncol (frame
  // by frame, so that every buffer holds items of all the tile's rows and all
  // four waves have work in every walk)
  const int nslot = nry * ntc * ncol;
  auto map_entry = [&](int s) -> int32_t {
    if (s >= nslot) return -1;
    const int k = s / ncol, c = s - k * ncol, x = xs + c;
    if (x < 0 || x >= W) return -1;
    const int yc = yc0 + k % nry, tc = t0 + k / nry;
    return bd.item_map[static_cast<int64_t>(tc) * C.HW + static_cast<int64_t>(yc) * W + x];
  };

  // Walks buffer entries 0 .. n - 1 in order.
  auto walk = [&](int n) {
    for (int i0 = 0; i0 < n; i0 += kWave) {
      const int ii = i0 + lane;
      const int2 entry = ii < n ? list[ii] : make_int2(0, 0);
      const int pp = entry.y;
      const int prow = pp >> 8, pcol = pp & 255;
      const int yc = yc0 + prow;
      // items out of reach of every lane of the wave are skipped (ballot)
      uint64_t m = __ballot(ii < n && yc >= wy0 - r && yc <= wy0 + 7 + r && pcol >= wc0 && pcol <= wc0 + 7 + 2 * r);
      while (m != 0) {
        const int bi = __ffsll(static_cast<unsigned long long>(m)) - 1;
        m &= m - 1;
        const int pu = __builtin_amdgcn_readlane(pp, bi);
        ScalarDouble* src = reinterpret_cast<ScalarDouble*>(reinterpret_cast<uintptr_t>(bd.rec)) +
                            static_cast<int64_t>(__builtin_amdgcn_readlane(entry.x, bi)) * R;
        double rc[R];
#pragma unroll
        for (int u = 0; u < R; ++u) rc[u] = src[u];
        const int dy = yq - (yc0 + (pu >> 8));
        const int dx = xq - (xs + (pu & 255));
        if (!in || dy < -r || dy > r || dx < -r || dx > r) continue;
        // the sample's regressors and weight (as the item's window pass forms
        // them, up to the rounding of the scaled features)
        const double vy = static_cast<double>(dy) * vy_step;
        const double kyy = K * vy;
        const double vx = static_cast<double>(dx) * vx_step;
        double v[F];
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          v[f] = fi[f] - rc[2 * P + 1 + f];
          if (f & 1) s1 = fma(v[f], v[f], s1);
          else s0 = fma(v[f], v[f], s0);
        }
        const double arg = fma(s0 + s1, K, fma(kyy, vy, K * vx * vx));
        const double w = static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(arg)));
        // (each operation takes one scalar operand)
        double cs = fma(rc[1], vx, rc[2] * vy) + rc[0];
        double pred = fma(rc[P + 1], vx, rc[P + 2] * vy) + rc[P];
#pragma unroll
        for (int f = 0; f < F; ++f) {
          cs = fma(rc[3 + f], v[f], cs);
          pred = fma(rc[P + 3 + f], v[f], pred);
        }
        acc = fma(w, cs, acc);
        const double kq = w * (cs * (yi - pred) - rc[2 * P]);
        gb[0] = fma(kq, vx * vx, gb[0]);
        gb[1] = fma(kq, vy * vy, gb[1]);
#pragma unroll
        for (int f = 0; f < F; ++f) gb[2 + f] = fma(kq, v[f] * v[f], gb[2 + f]);
      }
    }
  };

  // Steps of 256 slots fill the buffer; a walk empties it when a step's items
  // overflow it (the step is then resumed) and once after the last step.  One
  // walk site, so that the walk is compiled once.
  const int tid = static_cast<int>(threadIdx.x);
  int seq = 0;                                 // items of the region found so far (block-uniform)
  int base = 0;                                // sequence number of buffer entry 0
  int par = 0;
  int s = tid;                                 // this thread's first slot of the current step
  int32_t it[kGatherSlots];
  int mine[kGatherSlots];
  bool resume = false;
  int32_t next_it[kGatherSlots];
#pragma unroll
  for (int u = 0; u < kGatherSlots; ++u) {
    it[u] = -1;
    mine[u] = 0;
    next_it[u] = map_entry(s + u * kGatherThreads);
  }
  for (;;) {
    int nwalk = 0;                             // block-uniform
    const bool last = !resume && s - tid >= nslot;
    if (last) {
      nwalk = seq - base;
    } else {
      if (!resume) {
        int below[kGatherSlots];
#pragma unroll
        for (int u = 0; u < kGatherSlots; ++u) {
          it[u] = next_it[u];
          // in flight while this step is compacted and staged
          next_it[u] = map_entry(s + (kGatherSlots + u) * kGatherThreads);
          const uint64_t bal = __ballot(it[u] >= 0);
          below[u] = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(bal >> 32),
                                               __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(bal), 0));
          if (lane == 0) wcnt[(par * kGatherSlots + u) * kGatherWaves + wv] = __popcll(bal);
        }
        __syncthreads();                       // counts visible
#pragma unroll
        for (int u = 0; u < kGatherSlots; ++u) {
          int total = 0, off = 0;
#pragma unroll
          for (int w2 = 0; w2 < kGatherWaves; ++w2) {
            const int c = wcnt[(par * kGatherSlots + u) * kGatherWaves + w2];
            total += c;
            off += w2 < wv ? c : 0;
          }
          mine[u] = seq + off + below[u];
          seq += total;
        }
        par ^= 1;
      }
#pragma unroll
      for (int u = 0; u < kGatherSlots; ++u) {
        if (it[u] >= 0 && mine[u] >= base && mine[u] < base + cap) {
          const int su = s + u * kGatherThreads;
          const int k = su / ncol;
          list[mine[u] - base] = make_int2(it[u], ((k % nry) << 8) | (su - k * ncol));
        }
      }
      resume = seq > base + cap;
      if (resume) nwalk = cap;
      else s += kGatherSlots * kGatherThreads;
    }
    if (nwalk > 0) {
      __syncthreads();                         // the buffer is staged
      walk(nwalk);
      __syncthreads();                         // its reads are done
      base += nwalk;
    }
    if (last) break;
  }
  if (in && acc != 0.0) g_y[static_cast<int64_t>(tq) * C.HW + pq] += static_cast<float>(acc);
  // bandwidth partials of the block: a fixed butterfly inside each wave, then
  // the waves in order
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) gb[d] += __shfl_xor(gb[d], o);
  if (lane == 0)
#pragma unroll
    for (int d = 0; d < D; ++d) part[wv * D + d] = gb[d];
  __syncthreads();
  if (threadIdx.x < D) {
    double s = 0.0;
    for (int w2 = 0; w2 < kGatherWaves; ++w2) s += part[w2 * D + threadIdx.x];
    bd.gbpart[static_cast<int64_t>(blockIdx.x) * D + threadIdx.x] = s * C.sf[threadIdx.x] * C.h;
  }
}

template <int D>
__global__ void __launch_bounds__(256) reduce_gb_blocks(BwdDev bd) {
  __shared__ double sh[256][D];
  double acc[D];
#pragma unroll
  for (int d = 0; d < D; ++d) acc[d] = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < bd.npart;
       i += static_cast<int64_t>(gridDim.x) * 256)
#pragma unroll
    for (int d = 0; d < D; ++d) acc[d] += bd.gbpart[i * D + d];
#pragma unroll
  for (int d = 0; d < D; ++d) sh[threadIdx.x][d] = acc[d];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (static_cast<int>(threadIdx.x) < o)
#pragma unroll
      for (int d = 0; d < D; ++d) sh[threadIdx.x][d] += sh[threadIdx.x + o][d];
    __syncthreads();
  }
  if (threadIdx.x < D) bd.gbblk[blockIdx.x * D + threadIdx.x] = sh[0][threadIdx.x];
}

// One wave per bandwidth: lane l sums every 64th partial from the l-th on, then a
// fixed butterfly.
__global__ void __launch_bounds__(kWave* ESIM_MAX_D) reduce_gb_final(BwdDev bd, int nblk, int D, double* g_b) {
  const int d = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  double s = 0.0;
  for (int b = lane; b < nblk; b += kWave) s += bd.gbblk[b * D + d];
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) g_b[d] += s;
}

using GatherFn = void (*)(const ClipDev*, BwdDev, float*);

GatherFn pick_gather(int F) {
  switch (F) {
    case 1: return gather_kernel<1>;
    case 2: return gather_kernel<2>;
    case 3: return gather_kernel<3>;
    case 4: return gather_kernel<4>;
    case 5: return gather_kernel<5>;
    case 6: return gather_kernel<6>;
    case 7: return gather_kernel<7>;
    case 8: return gather_kernel<8>;
    case 9: return gather_kernel<9>;
    case 10: return gather_kernel<10>;
    case 11: return gather_kernel<11>;
    case 12: return gather_kernel<12>;
    default: return nullptr;
  }
}

using RedFn = void (*)(BwdDev);
template <int D>
RedFn red() { return reduce_gb_blocks<D>; }
RedFn pick_red(int D) {
  switch (D) {
    case 3: return red<3>();
    case 4: return red<4>();
    case 5: return red<5>();
    case 6: return red<6>();
    case 7: return red<7>();
    case 8: return red<8>();
    case 9: return red<9>();
    case 10: return red<10>();
    case 11: return red<11>();
    case 12: return red<12>();
    case 13: return red<13>();
    case 14: return red<14>();
    default: return nullptr;
  }
}

size_t align256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

int64_t gather_blocks(const ClipDev& hc) {
  return static_cast<int64_t>(hc.T) * ((hc.H + kGatherTile - 1) / kGatherTile) *
         ((hc.W + kGatherTile - 1) / kGatherTile);
}

struct Layout {
  size_t map, rec, gbpart, gbblk, total;
};

Layout layout(const ClipDev& hc, int64_t n) {
  Layout l{};
  const int D = hc.F + 2;
  size_t off = 0;
  l.map = off;
  off = align256(off + sizeof(int32_t) * static_cast<size_t>(hc.T) * hc.HW);
  l.rec = off;
  off = align256(off + sizeof(double) * adjoint_record(hc.F) * static_cast<size_t>(n));
  l.gbpart = off;
  off = align256(off + sizeof(double) * D * static_cast<size_t>(gather_blocks(hc)));
  l.gbblk = off;
  off = align256(off + sizeof(double) * kRedBlocks * D);
  l.total = off;
  return l;
}

unsigned grid_for(int64_t n, int64_t cap) {
  int64_t b = (n + 255) / 256;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

}  // namespace

size_t backward_scratch_bytes(const ClipDev& hc, int64_t n) { return layout(hc, n).total; }

hipError_t launch_backward(const BackwardArgs& a, hipStream_t s) {
  const ClipDev& hc = *a.host_clip;
  const int F = hc.F, D = F + 2;
  const RegressTable* t = regress_table(F);
  AdjointArgs adj{};
  adj.reg = a.reg;
  const AdjointFn fn = t ? t->adjoint[adj.reg.kind][hc.feat_f16 != 0] : nullptr;
  GatherFn gat = pick_gather(F);
  RedFn rb = pick_red(D);
  if (!fn || !gat || !rb) return hipErrorInvalidValue;
  const Layout l = layout(hc, a.n);
  char* m = static_cast<char*>(a.scratch);
  const int64_t gblocks = gather_blocks(hc);
  BwdDev bd{reinterpret_cast<int32_t*>(m + l.map), reinterpret_cast<double*>(m + l.rec),
            reinterpret_cast<double*>(m + l.gbpart), reinterpret_cast<double*>(m + l.gbblk), a.n, gblocks};
  const int64_t map_n = static_cast<int64_t>(hc.T) * hc.HW;
  hipLaunchKernelGGL(fill_map_kernel, dim3(grid_for(map_n, 4096)), dim3(256), 0, s, bd.item_map, map_n);
  hipLaunchKernelGGL(map_items_kernel, dim3(grid_for(a.n, 4096)), dim3(256), 0, s, a.clip, a.reg.items, a.n,
                     a.g_alpha, bd.item_map);
  adj.g_alpha = a.g_alpha;
  adj.bd = bd;
  adj.reg.max_groups = (a.n + kWave / 16 - 1) / (kWave / 16);
  const hipError_t e = launch_groups(reinterpret_cast<const void*>(fn), &adj, adj.reg, F, true, 1, a.dev, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gat, dim3(static_cast<unsigned>(gblocks)), dim3(kGatherThreads), 0, s, a.clip, bd, a.g_y);
  hipLaunchKernelGGL(rb, dim3(kRedBlocks), dim3(256), 0, s, bd);
  hipLaunchKernelGGL(reduce_gb_final, dim3(1), dim3(kWave * D), 0, s, bd, kRedBlocks, D, a.g_b);
  return hipGetLastError();
}

}  // namespace esim
