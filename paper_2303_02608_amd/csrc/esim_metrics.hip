// Nearest same-polarity neighbour distances between two event sets, for the
// event-set comparison of Sec. 3 (quantitative comparison: events as signed
// points (x, y, t); precision and recall count the events whose nearest
// same-polarity event of the other set lies within a threshold).
//
//   bitmap_clear_kernel  zero the occupancy bitmaps (a fill kernel, so a call
//                        can sit in a captured graph)
//   bitmap_set_kernel    one bit per source event in the bitmap of its
//                        polarity: [2][T][H][ceil(W / 32)] words (atomicOr:
//                        the result does not depend on the order)
//   nn_kernel            per query event: for the frames and rows of the box
//                        |dt| <= rt, |dy| <= ry, visited centre-out, the
//                        nearest set bit of the row within |dx| <= rx of the
//                        query column (count leading/trailing zeros over the
//                        row's words); the smallest scaled distance (FP64)
//                        wins, and rows whose (dt, dy) offset alone cannot beat
//                        it are not visited.  With rx, ry, rt the lattice
//                        extents of the radius rmax, this is the exact nearest
//                        neighbour within rmax.  nn_near_kernel: the same with
//                        the loads of two rows at a time in flight.
#include <cmath>
#include <cstdint>
#include <mutex>

#include "esim.h"
#include "esim_internal.h"

// Occupancy bitmaps of esim_nn_distances_noalloc: a fixed device array, so that
// call allocates nothing.  Each GPU the library runs on holds its own copy
// until the process ends.  In host code this name is a host-side stand-in, not
// a device address: the device address is obtained once per device with
// hipGetSymbolAddress (nn_static_scratch) and only that address is used.
static __device__ __align__(256) uint32_t scratch[ESIM_NN_STATIC_BYTES / sizeof(uint32_t)];

namespace esim {
namespace {

__global__ void __launch_bounds__(256) bitmap_clear_kernel(uint32_t* __restrict__ bm, int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) bm[i] = 0u;
}

__global__ void __launch_bounds__(256)
bitmap_set_kernel(uint32_t* __restrict__ bm, const int32_t* __restrict__ x, const int32_t* __restrict__ y,
                  const int32_t* __restrict__ t, const int8_t* __restrict__ p, int64_t n, int W, int H, int T,
                  int64_t wpr) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int xi = x[i], yi = y[i], ti = t[i], pi = p[i];
    if (xi < 0 || xi >= W || yi < 0 || yi >= H || ti < 0 || ti >= T || (pi != 1 && pi != -1)) continue;
    const int pl = pi > 0 ? 0 : 1;
    const int64_t w = ((static_cast<int64_t>(pl) * T + ti) * H + yi) * wpr + (xi >> 5);
    atomicOr(bm + w, 1u << (xi & 31));
  }
}

// Distance in columns from x to the nearest set bit of row within [lo, hi]
// (lo <= x <= hi), or -1 if none.
__device__ __forceinline__ int nearest_bit(const uint32_t* __restrict__ row, int x, int lo, int hi) {
  int best = -1;
  // right: lowest set bit in [x, hi]
  for (int w = x >> 5; w <= (hi >> 5); ++w) {
    uint32_t m = row[w];
    const int b0 = w << 5;
    if (b0 < x) m &= ~0u << (x - b0);
    if (b0 + 31 > hi) m &= (hi - b0 >= 31) ? ~0u : ((1u << (hi - b0 + 1)) - 1u);
    if (m) {
      best = b0 + __builtin_ctz(m) - x;
      break;
    }
  }
  // left: highest set bit in [lo, x - 1], only if it can be nearer
  const int lim = best < 0 ? x - lo : min(best - 1, x - lo);
  if (lim > 0) {
    const int l2 = x - lim;
    for (int w = (x - 1) >> 5; w >= (l2 >> 5); --w) {
      uint32_t m = row[w];
      const int b0 = w << 5;
      if (b0 + 31 > x - 1) m &= (x - 1 - b0 >= 31) ? ~0u : ((1u << (x - 1 - b0 + 1)) - 1u);
      if (b0 < l2) m &= ~0u << (l2 - b0);
      if (m) {
        const int d = x - (b0 + 31 - __builtin_clz(m));
        if (best < 0 || d < best) best = d;
        break;
      }
    }
  }
  return best;
}

constexpr uint32_t kOutside = 0xFFFFFFFCu;    // offset past any map: reads zero

__device__ __forceinline__ uint32_t ld_u32(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}

// The word of column x of a row with its two neighbours, and in them the distance
// to the nearest set bit within 32 columns of x (kNone if there is none).
struct RowWords {
  uint32_t before, at, after;
};
constexpr int kNone = 0x7fffffff;

__device__ __forceinline__ int nearest_of(const RowWords& r, int x) {
  const uint64_t here = (static_cast<uint64_t>(r.after) << 32) | r.at;
  const uint32_t b = static_cast<uint32_t>(x) & 31u;
  const uint64_t right = here >> b;                                       // bit i: column x + i
  const uint32_t left = static_cast<uint32_t>(((static_cast<uint64_t>(r.at) << 32) | r.before) >> b);   // x - 32 + i
  const uint32_t r1 = static_cast<uint32_t>(right >> 1);                  // bit i: column x + 1 + i
  const int dr = r1 ? 1 + __builtin_ctz(r1) : kNone;
  const int dl = left ? 1 + __builtin_clz(left) : kNone;
  return (right & 1u) ? 0 : min(dr, dl);
}

// nn_kernel for bitmaps below 4 GiB (offsets of a buffer resource).  A row is the
// three words around the query, those of the rows y - k and y + k go together, and
// the ones of k + 1 are in flight meanwhile; words further out are read only where
// these hold nothing and the box is wider.  Word by word and row by row, the
// search waited for each load before it knew the next.  1.5 and 3.45 million
// queries, 640 x 480 x 120, rmax 0.05: 126 and 384 us, now 50 and 137; the call for
// a million among 300000 in 1280 x 720 x 40 452, now 254; 200000 among 2000, rmax
// 0.1 (boxes of 257 x 145 x 9, nearly all empty) 5.2 ms, now 4.2.
__global__ void __launch_bounds__(256)
nn_near_kernel(const uint32_t* __restrict__ bm, uint32_t bytes, const int32_t* __restrict__ qx,
               const int32_t* __restrict__ qy, const int32_t* __restrict__ qt, const int8_t* __restrict__ qp,
               int64_t nq, int W, int H, int T, uint32_t wpr, double sx, double sy, double st, int rx, int ry, int rt,
               double rmax, double* __restrict__ d) {
  const __amdgpu_buffer_rsrc_t map = make_rsrc(bm, bytes);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nq; i += stride) {
    const int xi = qx[i], yi = qy[i], ti = qt[i], pi = qp[i];
    double best = INFINITY;
    if (xi >= 0 && xi < W && yi >= 0 && yi < H && ti >= 0 && ti < T && (pi == 1 || pi == -1)) {
      const uint32_t w0 = static_cast<uint32_t>(xi) >> 5;
      const bool first = w0 == 0, last = w0 + 1 == wpr;
      const int pl = pi > 0 ? 0 : 1;
      for (int kt = 0; kt <= 2 * rt; ++kt) {
        const int dt = (kt & 1) ? -((kt + 1) >> 1) : (kt >> 1);
        const double et = dt * st;
        if (et * et >= best) break;
        const int tc = ti + dt;
        if (tc < 0 || tc >= T) continue;
        const uint32_t frame = static_cast<uint32_t>(pl * T + tc) * static_cast<uint32_t>(H);
        auto row = [&](int yc) {
          const uint32_t at = ((frame + static_cast<uint32_t>(yc)) * wpr + w0) * 4u;
          // past the map's ends (rows outside the image, the word before the first) reads zero
          const bool in = static_cast<uint32_t>(yc) < static_cast<uint32_t>(H);
          RowWords r;
          r.before = ld_u32(map, in && !first ? at - 4u : kOutside);
          r.at = ld_u32(map, in ? at : kOutside);
          r.after = ld_u32(map, in && !last ? at + 4u : kOutside);
          return r;
        };
        // beyond 32 columns, two words at a time (s to the right and s to the left),
        // while they can hold a nearer bit of the box
        auto far = [&](int yc, double base) {
          const double e33 = 33.0 * sx;
          int dx = kNone;
          if (rx <= 32 || fma(e33, e33, base) >= best || yc < 0 || yc >= H) return dx;
          const uint32_t at = (frame + static_cast<uint32_t>(yc)) * wpr;
          const int b = xi & 31;
          for (int s = 1; 32 * s + min(-b, b - 31) <= min(rx, dx - 1); ++s) {
            const uint32_t wr = w0 + s, wl = w0 - s;           // (wl wraps past the row's start)
            const uint32_t mr = ld_u32(map, wr < wpr ? (at + wr) * 4u : kOutside);
            const uint32_t ml = ld_u32(map, wl < wpr ? (at + wl) * 4u : kOutside);
            if (mr) dx = min(dx, 32 * s - b + __builtin_ctz(mr));
            if (ml) dx = min(dx, 32 * s + b - 31 + __builtin_clz(ml));
          }
          return dx;
        };
        RowWords up = row(yi), down = up;
        for (int k = 0; k <= ry; ++k) {
          const double ey = k * sy;
          const double base = fma(et, et, ey * ey);
          if (base >= best) break;
          const RowWords u = up, v = down;
          if (k < ry) {
            up = row(yi - k - 1);
            down = row(yi + k + 1);
          }
          int dx = min(nearest_of(u, xi), nearest_of(v, xi));
          if (dx == kNone) dx = min(far(yi - k, base), k > 0 ? far(yi + k, base) : kNone);
          if (dx <= rx) {
            const double ex = dx * sx;
            best = min(best, fma(ex, ex, base));
          }
        }
      }
    }
    const double dist = sqrt(best);
    d[i] = dist <= rmax ? dist : INFINITY;
  }
}

__global__ void __launch_bounds__(256)
nn_kernel(const uint32_t* __restrict__ bm, const int32_t* __restrict__ qx, const int32_t* __restrict__ qy,
          const int32_t* __restrict__ qt, const int8_t* __restrict__ qp, int64_t nq, int W, int H, int T,
          int64_t wpr, double sx, double sy, double st, int rx, int ry, int rt, double rmax,
          double* __restrict__ d) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < nq; i += stride) {
    const int xi = qx[i], yi = qy[i], ti = qt[i], pi = qp[i];
    double best = INFINITY;
    if (xi >= 0 && xi < W && yi >= 0 && yi < H && ti >= 0 && ti < T && (pi == 1 || pi == -1)) {
      const int pl = pi > 0 ? 0 : 1;
      const int lo = max(0, xi - rx), hi = min(W - 1, xi + rx);
      // frames and rows centre-out (0, -1, +1, -2, +2, ...): |dt| and |dy| never
      // decrease, so once a row's offset alone reaches the best distance every
      // later row of the frame (and, at dy = 0, every later frame) does too
      for (int kt = 0; kt <= 2 * rt; ++kt) {
        const int dt = (kt & 1) ? -((kt + 1) >> 1) : (kt >> 1);
        const double et = dt * st;
        if (et * et >= best) break;
        const int tc = ti + dt;
        if (tc < 0 || tc >= T) continue;
        for (int ky = 0; ky <= 2 * ry; ++ky) {
          const int dy = (ky & 1) ? -((ky + 1) >> 1) : (ky >> 1);
          const double ey = dy * sy;
          const double base = fma(et, et, ey * ey);
          if (base >= best) break;
          const int yc = yi + dy;
          if (yc < 0 || yc >= H) continue;
          const uint32_t* row = bm + ((static_cast<int64_t>(pl) * T + tc) * H + yc) * wpr;
          const int dx = nearest_bit(row, xi, lo, hi);
          if (dx >= 0) {
            const double ex = dx * sx;
            best = min(best, fma(ex, ex, base));
          }
        }
      }
    }
    const double dist = sqrt(best);
    d[i] = dist <= rmax ? dist : INFINITY;
  }
}

unsigned grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

}  // namespace

bool nn_static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return false;
    addr[dev] = p;
  }
  *out = addr[dev];
  return true;
}

size_t nn_scratch_bytes(int W, int H, int T) {
  const int64_t wpr = (static_cast<int64_t>(W) + 31) / 32;
  return sizeof(uint32_t) * 2 * static_cast<size_t>(T) * H * wpr;
}

hipError_t launch_nn(const NnArgs& a, hipStream_t s) {
  const int64_t wpr = (static_cast<int64_t>(a.W) + 31) / 32;
  const int64_t words = 2 * static_cast<int64_t>(a.T) * a.H * wpr;
  uint32_t* bm = static_cast<uint32_t*>(a.scratch);
  hipLaunchKernelGGL(bitmap_clear_kernel, dim3(grid_for(words)), dim3(256), 0, s, bm, words);
  if (a.ns > 0)
    hipLaunchKernelGGL(bitmap_set_kernel, dim3(grid_for(a.ns)), dim3(256), 0, s, bm, a.sx, a.sy, a.st, a.sp,
                       a.ns, a.W, a.H, a.T, wpr);
  if (a.nq > 0 && words * 4 < (static_cast<int64_t>(1) << 32) - 4)
    hipLaunchKernelGGL(nn_near_kernel, dim3(grid_for(a.nq)), dim3(256), 0, s, bm, static_cast<uint32_t>(words * 4), a.qx,
                       a.qy, a.qt, a.qp, a.nq, a.W, a.H, a.T, static_cast<uint32_t>(wpr), a.scale_x, a.scale_y,
                       a.scale_t, a.rx, a.ry, a.rt, a.rmax, a.d);
  else if (a.nq > 0)
    hipLaunchKernelGGL(nn_kernel, dim3(grid_for(a.nq)), dim3(256), 0, s, bm, a.qx, a.qy, a.qt, a.qp, a.nq, a.W,
                       a.H, a.T, wpr, a.scale_x, a.scale_y, a.scale_t, a.rx, a.ry, a.rt, a.rmax, a.d);
  return hipGetLastError();
}

}  // namespace esim
