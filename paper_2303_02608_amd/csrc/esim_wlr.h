// Window geometry, window walks, lane sums and solve of one weighted local
// regression (Sec. 2.1, eqs. 4-5), shared by the forward, bandwidth and adjoint
// kernels.
//
// Regressors are kept in bandwidth-scaled units v_j = u_j / (h b_j): the
// weight exponent is then sum_j v_j^2 (eq. 5 with a Gaussian fall-off) and
// the fit in v equals the fit in u with beta_j = theta_j / (h b_j) and the
// ridge scaled to lambda / (h b_j)^2.
//
// The FP64 Gram's walks: walk_frames (columns of a lane, read from memory, for
// lists, small frames and windows beyond LDS) and tile_frames (a pixel per lane,
// windows from LDS, for whole frames).  window_loop is the older loop of the compensated FP32 Gram, whose
// rounding depends on its order, and of the explicit threshold: the L lanes of an
// item split the window columns (lane j takes dx = -r + j, -r + j + L, ...), and
// the rows (dt, dy) of a column are software-pipelined in registers, loaded two
// rows ahead of their use.  Rows outside the image (or past the last row) read the
// valid centre pixel and get weight 0.
#pragma once

#include <type_traits>

#include "esim_internal.h"

namespace esim {

constexpr double kHalfLog2e = -0.72134752044448170368;  // -log2(e) / 2

template <int F, bool F16, class Real = double>
struct ItemGeom {
  static constexpr uint32_t ES = F16 ? 2u : 4u;
  __amdgpu_buffer_rsrc_t ry, rf;
  uint32_t HW, vcen_f, vcen_y;
  int W, H, T, r, tr, px, py, fc, tt, dt_lo, dt_hi;
  bool active;
  Real sf[F + 2];
  Real xcs[F];
  Real vx_step, vy_step;
};

// Fills the geometry of the item at (pix, tt) of clip C.  f0/f1 are the frames
// the buffer resources cover (a uniform frame's window, or the whole clip).
template <int F, bool F16, class Real>
__device__ __forceinline__ void make_geom(ItemGeom<F, F16, Real>& g, const ClipDev& C, int64_t pix,
                                          int tt, int f0, int f1, bool active) {
  constexpr uint32_t ES = ItemGeom<F, F16, Real>::ES;
  g.W = C.W;
  g.H = C.H;
  g.T = C.T;
  g.r = C.r;
  g.tr = C.tr;
  g.HW = static_cast<uint32_t>(C.HW);
  g.active = active;
  g.tt = tt;
  g.ry = make_rsrc(C.y + static_cast<uint64_t>(f0) * g.HW, static_cast<uint64_t>(f1 - f0) * g.HW * 4u);
  g.rf = make_rsrc(static_cast<const char*>(C.feat) + static_cast<uint64_t>(f0) * F * g.HW * ES,
                   static_cast<uint64_t>(f1 - f0) * F * g.HW * ES);
  g.py = static_cast<int>(pix / g.W);
  g.px = static_cast<int>(pix - static_cast<int64_t>(g.py) * g.W);
  g.fc = tt - f0;
  g.vcen_f = (static_cast<uint32_t>(g.fc) * F * g.HW + static_cast<uint32_t>(pix)) * ES;
  g.vcen_y = (static_cast<uint32_t>(g.fc) * g.HW + static_cast<uint32_t>(pix)) * 4u;
#pragma unroll
  for (int d = 0; d < F + 2; ++d) g.sf[d] = static_cast<Real>(C.sf[d]);
#pragma unroll
  for (int f = 0; f < F; ++f)
    g.xcs[f] = static_cast<Real>(ld_feat<F16>(g.rf, g.vcen_f, f * g.HW * ES)) * g.sf[2 + f];
  g.vx_step = static_cast<Real>(C.sf[0] / g.r);
  g.vy_step = static_cast<Real>(C.sf[1] / g.r);
  g.dt_lo = max(-g.tr, -tt);
  g.dt_hi = min(g.tr, g.T - 1 - tt);
}

// Runs the window of one item in lane j of its L-lane group.
//   pass_begin(vx)                      before each column pass
//   sample(w, yd, v[F], vy, dx, dt, dy, ok) for every row of the window in
//                                       the lane's column; ok is false (and
//                                       w = 0) outside the image and for idle
//                                       columns
//   pass_end(vx)                        after each column pass
//
// The rows of a column form a three-stage software pipeline: the loads of row
// k+2 are in flight while the weight of row k+1 is computed and row k is
// accumulated, so the exponential's latency overlaps independent Gram work.
// The loop takes two rows per iteration (see the loop for an odd row count).
// Row offsets advance by uniform (SGPR) amounts; only the validity test and
// the select are per lane.
template <int F, int L, bool F16, class Real, class PassBegin, class Sample, class PassEnd>
__device__ __forceinline__ void window_loop(const ItemGeom<F, F16, Real>& g, int j,
                                            PassBegin&& pass_begin, Sample&& sample,
                                            PassEnd&& pass_end) {
  constexpr uint32_t ES = ItemGeom<F, F16, Real>::ES;
  constexpr Real K = static_cast<Real>(kHalfLog2e);
  const int r = g.r;
  const int span = 2 * r + 1;
  const int nt = g.dt_hi - g.dt_lo + 1;
  const int nrows = nt * span;
  const int npass = (span + L - 1) / L;
  // per-lane valid row range of the item (rows inside the image)
  const int dy_lo = -min(r, g.py), dy_hi = min(r, g.H - 1 - g.py);
  const uint32_t WES = static_cast<uint32_t>(g.W) * ES, W4 = static_cast<uint32_t>(g.W) * 4u;
  const uint32_t FES = static_cast<uint32_t>(F) * g.HW * ES, HW4 = g.HW * 4u;
  for (int k = 0; k < npass; ++k) {
    const int dx = -r + j + k * L;
    const int col = g.px + dx;
    const bool col_ok = g.active && dx <= r && col >= 0 && col < g.W;
    const Real vx = static_cast<Real>(dx) * g.vx_step;
    const Real kx = K * vx * vx;
    pass_begin(vx);
    // offsets of the window's first row (dt_lo, -r) in this column; rows above
    // the image wrap as unsigned and are never used (the select takes the
    // centre instead)
    const uint32_t vf_base = (static_cast<uint32_t>(g.fc + g.dt_lo) * F * g.HW +
                              static_cast<uint32_t>((g.py - r) * g.W + col)) * ES;
    const uint32_t vy_base = (static_cast<uint32_t>(g.fc + g.dt_lo) * g.HW +
                              static_cast<uint32_t>((g.py - r) * g.W + col)) * 4u;
    int ldt = 0, ldy = 0;          // next row to load, relative to (dt_lo, -r)
    auto load_row = [&](float& yv, float (&fv)[F]) -> bool {
      const int dy = ldy - r;
      const bool ok = (ldt <= g.dt_hi - g.dt_lo) & col_ok & (dy >= dy_lo) & (dy <= dy_hi);
      const uint32_t sof = static_cast<uint32_t>(ldt) * FES + static_cast<uint32_t>(ldy) * WES;
      const uint32_t soy = static_cast<uint32_t>(ldt) * HW4 + static_cast<uint32_t>(ldy) * W4;
      const uint32_t vf = ok ? vf_base + sof : g.vcen_f;
      const uint32_t vy = ok ? vy_base + soy : g.vcen_y;
      yv = ld_f32(g.ry, vy, 0);
#pragma unroll
      for (int f = 0; f < F; ++f) fv[f] = ld_feat<F16>(g.rf, vf, f * g.HW * ES);
      if (++ldy == span) {
        ldy = 0;
        ++ldt;
      }
      return ok;
    };
    struct Wt {
      Real w, yd, vy, v[F];
      int dt, dy;
      bool ok;
    };
    int cdt = g.dt_lo, cdy = -r;   // next row to weigh
    auto weigh = [&](float yv, const float (&fv)[F], bool ok, Wt& o) {
      o.dy = cdy;
      o.dt = cdt;
      o.ok = ok;
      if (++cdy > r) {
        cdy = -r;
        ++cdt;
      }
      o.vy = static_cast<Real>(o.dy) * g.vy_step;
      Real s0 = 0, s1 = 0;
#pragma unroll
      for (int f = 0; f < F; ++f) {
        o.v[f] = fma(static_cast<Real>(fv[f]), g.sf[2 + f], -g.xcs[f]);
        if (f & 1) s1 = fma(o.v[f], o.v[f], s1);
        else s0 = fma(o.v[f], o.v[f], s0);
      }
      const Real arg = fma(s0 + s1, K, fma(K * o.vy, o.vy, kx));
      const float e = __builtin_amdgcn_exp2f(static_cast<float>(arg));
      o.w = static_cast<Real>(ok ? e : 0.0f);
      o.yd = static_cast<Real>(yv);
    };
    auto use = [&](const Wt& o) { sample(o.w, o.yd, o.v, o.vy, dx, o.dt, o.dy, o.ok); };
    // pipeline prologue: rows 0 and 1 loaded, row 0 weighed, row 2 in flight
    float yA, fA[F], yB, fB[F];
    bool okA = load_row(yA, fA);
    bool okB = load_row(yB, fB) & (1 < nrows);
    Wt wA, wB;
    weigh(yA, fA, okA, wA);
    okA = load_row(yA, fA) & (2 < nrows);
    // FP64: pairs of rows, then an odd last row alone.  FP32 (the compensated
    // variant, whose per-sample body is larger): pairs only, an odd count
    // ending on a weight-0 padding row, which measured faster there.
    constexpr bool kPeel = std::is_same<Real, double>::value;
    const int qend = kPeel ? nrows - 1 : nrows;
    int q = 0;
#pragma unroll 1
    for (; q < qend; q += 2) {
      // wA = row q (weighed), raw B = row q+1, raw A = row q+2
      weigh(yB, fB, okB, wB);
      okB = load_row(yB, fB) & (q + 3 < nrows);
      use(wA);
      weigh(yA, fA, okA, wA);
      okA = load_row(yA, fA) & (q + 4 < nrows);
      use(wB);
    }
    if constexpr (kPeel) {
      if (q < nrows) use(wA);     // odd row count: the last row alone
    }
    pass_end(vx);
  }
}

// ---- the column walk of the FP64 regression -------------------------------
//
// One lane owns one column of an item's window at a time and walks its rows
// from dy = -r to r, the frames of a row innermost, so that both coordinates
// are constant over the 2 tr + 1 samples of a cell (dx, dy).  No entry with a
// coordinate factor is summed per sample:
//   v_x  constant in the column: a factor of the column's sums;
//   v_y  CellSums: a cell's (w, w y, w f) are summed by themselves and go, once per
//        cell, to the column's sums and, times the row, to its moments;
//        RunSums: the running column sums C_k after cell k are added up once per
//        cell, P = sum_k C_k; a cell at dy, e rows before the walk's end, is then
//        counted e - dy times, so sum dy s = e C - P, and with PP = sum_k P_k
//        sum dy^2 s = e^2 C - (2 e + 1) P + 2 PP.
// A cell at tr = 1 and F = 7 spends 19 instructions there less the 9 adds that its
// first sample saves (CellSums), or 10 adds, where one row of samples at a time
// spent 11 fused multiply-adds and a multiply per sample.
//
// CellSums round a moment to 2^-53 or so of itself.  RunSums let the centre row's
// weight, up to the whole of W, cancel to zero: a moment (of the W-normalised,
// bandwidth-scaled system) keeps an error of about 4e-16 / (h b)^2.  That is the
// ridge's own scale: it acts as a ridge changed by 4e-16.  The dense walks take
// CellSums, which cost them nothing; in the lists' 256 registers the cell's own sums
// cost 10 % (F = 7, r = 7, 100 000 items 250 -> 277 us, 2000 items 18 -> 23), so they
// take RunSums unless the ridge is small (kExactRidge).
//
// Samples outside the image read the nearest pixel inside it, which lies in
// the window too (so a NaN there counts where it counts anyway), and get
// weight 0 through an exponent of kDropped.  Frames outside the clip are not
// walked: the caller passes lanes whose items share dt_lo and nt.

constexpr double kDropped = -65536.0;    // exponent (base 2) of a sample of weight 0

// Sums of products without a coordinate, over all of a lane's samples.
template <int F>
struct ProductSums {
  static constexpr int NA = F * (F + 1) / 2;
  double Syy, gf[F], Aff[NA];

  __device__ __forceinline__ void zero() {
    Syy = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) gf[k] = 0;
#pragma unroll
    for (int k = 0; k < NA; ++k) Aff[k] = 0;
  }
  // Adds a sample; sink(k, wz) takes w y (k = -1) and w f_k.
  template <class Sink>
  __device__ __forceinline__ void add(double w, double yd, const double (&v)[F], Sink&& sink) {
    const double wy = w * yd;
    sink(-1, wy);
    Syy = fma(wy, yd, Syy);
    int q = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) {
      const double wz = w * v[k];
      sink(k, wz);
      gf[k] = fma(wz, yd, gf[k]);
#pragma unroll
      for (int e = k; e < F; ++e) {
        Aff[q] = fma(wz, v[e], Aff[q]);
        ++q;
      }
    }
  }
};

template <int F>
struct CellSums {
  double cW, cg, cf[F];            // of the cell: w, w y, w f
  double W, g, f[F], YW;           // of the line, and the first moment of w along it
  double YY, Yg, Yf[F];            // of all lines: the second moment of w, the first of w y, w f
  ProductSums<F> p;

  __device__ __forceinline__ void zero() {
    W = g = YW = YY = Yg = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) f[k] = Yf[k] = 0;
    p.zero();
  }
  // A sample; `first` of its cell (a constant after unrolling).
  __device__ __forceinline__ void add(double w, double yd, const double (&v)[F], bool first) {
    cW = first ? w : cW + w;
    p.add(w, yd, v, [&](int k, double wz) {
      double& c = k < 0 ? cg : cf[k < 0 ? 0 : k];
      c = first ? wz : c + wz;
    });
  }
  // The cell at d along the line is complete.
  __device__ __forceinline__ void end_cell(int di) {
    const double d = static_cast<double>(di), dW = d * cW;
    W += cW;
    YW += dW;
    YY = fma(d, dW, YY);
    g += cg;
    Yg = fma(d, cg, Yg);
#pragma unroll
    for (int k = 0; k < F; ++k) {
      f[k] += cf[k];
      Yf[k] = fma(d, cf[k], Yf[k]);
    }
  }
};

template <int F>
struct RunSums {
  double W, g, f[F];               // running sums of w, w y, w f
  double PW, Pg, Pf[F], PPW;       // their sums over the cells, and the sums of PW
  ProductSums<F> p;

  __device__ __forceinline__ void zero() {
    W = g = PW = Pg = PPW = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) f[k] = Pf[k] = 0;
    p.zero();
  }
  __device__ __forceinline__ void add(double w, double yd, const double (&v)[F], bool) {
    W += w;
    p.add(w, yd, v, [&](int k, double wz) { (k < 0 ? g : f[k < 0 ? 0 : k]) += wz; });
  }
  __device__ __forceinline__ void end_cell(int) {
    PW += W;
    PPW += PW;
    Pg += g;
#pragma unroll
    for (int k = 0; k < F; ++k) Pf[k] += f[k];
  }
};

// What the finished lines of a lane add up to: the sums, and the lines' coordinate
// (X) times them; YW as in CellSums, XY its moment with the lines' coordinate.
template <int F>
struct LaneSums {
  double W, g, f[F], YW;
  double XW, XX, Xg, Xf[F], XY;

  __device__ __forceinline__ void zero() {
    W = g = YW = XW = Xg = XX = XY = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) f[k] = Xf[k] = 0;
  }
  // Takes over the line at coordinate x and clears its part of c (the sums
  // without a line's coordinate stay in c).
  __device__ __forceinline__ void end_line(CellSums<F>& c, double x) {
    W += c.W;
    XW = fma(x, c.W, XW);
    XX = fma(x * x, c.W, XX);
    YW += c.YW;
    XY = fma(x, c.YW, XY);
    g += c.g;
    Xg = fma(x, c.g, Xg);
    c.W = c.g = c.YW = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) {
      f[k] += c.f[k];
      Xf[k] = fma(x, c.f[k], Xf[k]);
      c.f[k] = 0;
    }
  }
};

// Geometry of the column walk of one lane's item.
template <int F, bool F16>
struct WalkGeom {
  static constexpr uint32_t ES = F16 ? 2u : 4u;
  __amdgpu_buffer_rsrc_t ry, rf;
  uint32_t HW;
  uint32_t vf0, vy0;               // byte offsets of (frame tt + dt_lo, row max(py - r, 0), column 0)
  int W, H, r, nt, px, py;
  bool active;
  double sf[F], xcs[F];
  double vx_step, vy_step;
  double kexp;                     // the exponent (base 2) of a weight is kexp |v|^2
};

// Fills the geometry of the item at (pix, tt) of clip C, whose window holds the
// nt frames from tt + dt_lo on.  f0/f1 are the frames the buffer resources cover
// (a uniform frame's window, or the whole clip).  wscale scales the weights'
// exponent.
template <int F, bool F16>
__device__ __forceinline__ void make_walk(WalkGeom<F, F16>& g, const ClipDev& C, int64_t pix, int tt, int dt_lo,
                                          int nt, int f0, int f1, bool active, double wscale = 1.0) {
  constexpr uint32_t ES = WalkGeom<F, F16>::ES;
  g.W = uni(C.W);
  g.H = uni(C.H);
  g.r = uni(C.r);
  g.nt = nt;
  g.HW = static_cast<uint32_t>(uni(static_cast<int>(C.HW)));
  g.active = active;
  g.ry = make_rsrc(uni(C.y) + static_cast<uint64_t>(f0) * g.HW, static_cast<uint64_t>(f1 - f0) * g.HW * 4u);
  g.rf = make_rsrc(static_cast<const char*>(uni(C.feat)) + static_cast<uint64_t>(f0) * F * g.HW * ES,
                   static_cast<uint64_t>(f1 - f0) * F * g.HW * ES);
  const uint32_t up = static_cast<uint32_t>(pix), uw = static_cast<uint32_t>(g.W);
  g.py = static_cast<int>(up / uw);
  g.px = static_cast<int>(up - static_cast<uint32_t>(g.py) * uw);
  const uint32_t fc = static_cast<uint32_t>(tt - f0);
  const uint32_t fl = static_cast<uint32_t>(tt + dt_lo - f0);
  const uint32_t row0 = static_cast<uint32_t>(max(g.py - g.r, 0)) * uw;
  g.vf0 = (fl * F * g.HW + row0) * ES;
  g.vy0 = (fl * g.HW + row0) * 4u;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    g.sf[f] = uni(C.sf[2 + f]);
    g.xcs[f] = static_cast<double>(ld_feat<F16>(g.rf, (fc * F * g.HW + up) * ES, f * g.HW * ES)) * g.sf[f];
  }
  g.vx_step = C.sf[0] / g.r;
  g.vy_step = C.sf[1] / g.r;
  g.kexp = kHalfLog2e * wscale;
}

// Walks R consecutive frames, the first k0 frames after dt_lo, of the column dx
// of the lane's item (dx > r: an idle column, weight 0), adding their samples to
// c.  DEPTH (1 or 2) cells of samples are loaded ahead: a sample's registers are
// reloaded as soon as it is used.  PART: only the n rows from s0 on (s0 >= -r may
// differ between the lanes; rows below r get weight 0).
template <int F, bool F16, int R, int DEPTH = 1, bool PART = false, class Sums>
__device__ __forceinline__ void walk_frames(const WalkGeom<F, F16>& g, int dx, int k0, Sums& c,
                                            int s0 = 0, int n = 0) {
  constexpr uint32_t ES = WalkGeom<F, F16>::ES;
  const double K = g.kexp;
  const int r = g.r;
  const int col = g.px + dx;
  const bool col_ok = g.active && dx <= r && static_cast<uint32_t>(col) < static_cast<uint32_t>(g.W);
  const uint32_t cc = static_cast<uint32_t>(min(max(g.px + min(dx, r), 0), g.W - 1));
  const double vx = static_cast<double>(dx) * g.vx_step;
  const double kx = col_ok ? K * vx * vx : kDropped;
  const double kyy = K * g.vy_step * g.vy_step;
  const uint32_t WES = static_cast<uint32_t>(g.W) * ES, W4 = static_cast<uint32_t>(g.W) * 4u;
  const uint32_t HES = g.HW * ES, FES = static_cast<uint32_t>(F) * HES, HW4 = g.HW * 4u;
  const uint32_t sof = static_cast<uint32_t>(k0) * FES, soy = static_cast<uint32_t>(k0) * HW4;   // uniform
  uint32_t vf = g.vf0 + cc * ES, vy = g.vy0 + cc * 4u;         // offsets of the next row to load
  if constexpr (PART) {                    // from row py + s0 on
    const uint32_t skip = static_cast<uint32_t>(min(max(g.py + min(s0, r), 0), g.H - 1) - max(g.py - r, 0));
    vf += skip * WES;
    vy += skip * W4;
  }
  float ys[DEPTH][R];
  Feat<F16> fs[DEPTH][R][F];
  auto load = [&](int d, int i) {
    ys[d][i] = ld_f32(g.ry, vy, soy + i * HW4);
#pragma unroll
    for (int f = 0; f < F; ++f) fs[d][i][f] = ld_raw<F16>(g.rf, vf, sof + i * FES + f * HES);
  };
  auto next_row = [&](int dy) {            // a step down where rows dy and dy + 1 are in the image
                                           // (a part's also in the window: what it reads counts)
    const bool down = static_cast<uint32_t>(g.py + dy) < static_cast<uint32_t>(g.H - 1) && (!PART || dy < r);
    vf += down ? WES : 0u;
    vy += down ? W4 : 0u;
  };
  auto cell = [&](int d, int dy) {
    next_row(dy + DEPTH - 1);
    const double e = fma(kyy, static_cast<double>(dy * dy), kx);
    const bool row_ok = static_cast<uint32_t>(g.py + dy) < static_cast<uint32_t>(g.H) && (!PART || dy <= r);
    const double base = row_ok ? e : kDropped;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      double v[F], s0 = 0, s1 = 0;
#pragma unroll
      for (int f = 0; f < F; ++f) {
        v[f] = fma(static_cast<double>(feat_f32(fs[d][i][f])), g.sf[f], -g.xcs[f]);
        if (f & 1) s1 = fma(v[f], v[f], s1);
        else s0 = fma(v[f], v[f], s0);
      }
      const double arg = fma(s0 + s1, K, base);
      const double w = static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(arg)));
      const double yd = static_cast<double>(ys[d][i]);
      load(d, i);
      c.add(w, yd, v, i == 0);
    }
    c.end_cell(dy);
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
    for (int i = 0; i < R; ++i) load(d, i);
    if (d + 1 < DEPTH) next_row(d + (PART ? s0 : -r));
  }
  if constexpr (PART && DEPTH == 1) {
#pragma unroll 1
    for (int k = 0; k < n; ++k) cell(0, s0 + k);
  } else if constexpr (PART) {
#pragma unroll 1
    for (int k = 0; k + 1 < n; k += 2) {
      cell(0, s0 + k);
      cell(1, s0 + k + 1);
    }
    if (n & 1) cell(0, s0 + n - 1);
  } else if constexpr (DEPTH == 1) {
#pragma unroll 1
    for (int dy = -r; dy <= r; ++dy) cell(0, dy);
  } else {
    // 2 r + 1 rows: pairs, and the last one
#pragma unroll 1
    for (int dy = -r; dy < r; dy += 2) {
      cell(0, dy);
      cell(1, dy + 1);
    }
    cell(0, r);
  }
}

// ---- dense windows from LDS ------------------------------------------------
//
// Every pixel of a frame, one lane per pixel: a wave owns a tile of 64 pixels
// (64 x 1, 32 x 2 or 16 x 4) and keeps the rows of the window that its pixels are
// reading in its own LDS, one record of all channels per pixel: (frames of a
// cell) x (features and y), single precision, in 16-byte units.  A lane walks its
// window row by row, so a step of the walk is one record further; the walked
// coordinate of CellSums is v_x here and the lines' one is v_y.  The rows are a
// ring as high as the tile; a new row replaces the one that left.
//
// Read straight from memory, a sample is 8 loads at F = 7, and 64 lanes' window
// rows do not stay in the L1: every column pass fetched its 90 KB from L2 again,
// 12 cycles a load of the CU's one vector memory path, so that the four SIMDs' 32
// loads a sample took longer than the 87 VALU instructions beside them.  From LDS a
// sample is two 16-byte reads, and memory is read once per row.  Records have an
// odd number of units, so that neighbouring lanes' reads fall on different banks.
//
// The tile is a wave's and not a block's so that no wave waits at a barrier: a
// SIMD issues its older wave first, which takes three of four issue slots, and
// the younger one the rest.  Waves that keep step at barriers, or that are given
// equal shares, leave the younger ones to run alone for half of the launch, at the
// 5.5 cycles a VALU instruction that one wave reaches; waves that fetch their next
// tile when they are done fill the slots to the end (see GroupQueue).

// One tile of one clip at frame tt.
template <int F, bool F16>
struct TileGeom {
  static constexpr uint32_t ES = F16 ? 2u : 4u;
  __amdgpu_buffer_rsrc_t ry, rf;
  uint32_t HW;
  int W, H, r, nt, lw;             // tile width 2^lw
  int x0, y0;                      // the tile's first pixel
  int px, py;                      // this lane's pixel (may lie outside the image)
  double sf[F], xcs[F];
  double vx_step, vy_step;
  double kexp;                     // the exponent (base 2) of a weight is kexp |v|^2
};

template <int F, bool F16>
__device__ __forceinline__ void make_tile(TileGeom<F, F16>& g, const ClipDev& C, int tile, int tt,
                                          double wscale = 1.0) {
  constexpr uint32_t ES = TileGeom<F, F16>::ES;
  const int lane = threadIdx.x & (kWave - 1);
  g.W = uni(C.W);
  g.H = uni(C.H);
  g.r = uni(C.r);
  g.lw = uni(C.tile_lw);
  g.HW = static_cast<uint32_t>(uni(static_cast<int>(C.HW)));
  const int tr = uni(C.tr), T = uni(C.T);
  const int f0 = max(0, tt - tr), f1 = min(T, tt + tr + 1);
  g.nt = f1 - f0;
  g.ry = make_rsrc(uni(C.y) + static_cast<uint64_t>(f0) * g.HW, static_cast<uint64_t>(f1 - f0) * g.HW * 4u);
  g.rf = make_rsrc(static_cast<const char*>(uni(C.feat)) + static_cast<uint64_t>(f0) * F * g.HW * ES,
                   static_cast<uint64_t>(f1 - f0) * F * g.HW * ES);
  const int ntx = (g.W + (1 << g.lw) - 1) >> g.lw;
  const int ty = tile / ntx;
  g.x0 = (tile - ty * ntx) << g.lw;
  g.y0 = ty * (kWave >> g.lw);
  g.px = g.x0 + (lane & ((1 << g.lw) - 1));
  g.py = g.y0 + (lane >> g.lw);
  const uint32_t cen = static_cast<uint32_t>(min(g.py, g.H - 1)) * static_cast<uint32_t>(g.W) +
                       static_cast<uint32_t>(min(g.px, g.W - 1));
#pragma unroll
  for (int f = 0; f < F; ++f) {
    g.sf[f] = uni(C.sf[2 + f]);
    g.xcs[f] = static_cast<double>(ld_feat<F16>(g.rf, (static_cast<uint32_t>(tt - f0) * F * g.HW + cen) * ES,
                                                f * g.HW * ES)) * g.sf[f];
  }
  g.vx_step = C.sf[0] / g.r;
  g.vy_step = C.sf[1] / g.r;
  g.kexp = kHalfLog2e * wscale;
}

// Orders a wave's LDS accesses before and after it (between lanes of the wave:
// the hardware runs a wave's LDS instructions in order, the compiler must too).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// Row y of the image on its way to a ring slot: frames k0 .. k0 + R - 1 of the
// window, columns x0 - r .. x0 + 2^lw + r - 1 (at most 2 kWave), row and columns
// clamped to the image.  load issues the loads of turn h of the wave's lanes,
// store writes them to LDS.
template <int F, bool F16, int R>
struct RowLoads {
  static constexpr uint32_t ES = TileGeom<F, F16>::ES;
  static constexpr int NQ = tile_quads(F), U = tile_units(F, R);
  Feat<F16> v[R][F];
  float y[R];

  __device__ __forceinline__ void load(const TileGeom<F, F16>& g, int h, int y0, int k0) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t row = static_cast<uint32_t>(min(max(y0, 0), g.H - 1)) * static_cast<uint32_t>(g.W);
    const uint32_t x = static_cast<uint32_t>(min(max(g.x0 - g.r + lane + h * kWave, 0), g.W - 1));
#pragma unroll
    for (int i = 0; i < R; ++i) {
#pragma unroll
      for (int c = 0; c < F; ++c)
        v[i][c] = ld_raw<F16>(g.rf, x * ES, (static_cast<uint32_t>((k0 + i) * F + c) * g.HW + row) * ES);
      y[i] = ld_f32(g.ry, x * 4u, (static_cast<uint32_t>(k0 + i) * g.HW + row) * 4u);
    }
  }
  __device__ __forceinline__ void store(const TileGeom<F, F16>& g, float4* lds, int h, int slot) const {
    const int p = static_cast<int>(threadIdx.x & (kWave - 1)) + h * kWave;
    const int rowpx = (1 << g.lw) + 2 * g.r;
    if (p < rowpx) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        float ch[4 * NQ] = {};
#pragma unroll
        for (int c = 0; c < F; ++c) ch[c] = feat_f32(v[i][c]);
        ch[F] = y[i];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          lds[(slot * rowpx + p) * U + i * NQ + q] =
              make_float4(ch[4 * q], ch[4 * q + 1], ch[4 * q + 2], ch[4 * q + 3]);
      }
    }
  }
};

template <int F, bool F16, int R>
__device__ __forceinline__ void stage_row(const TileGeom<F, F16>& g, float4* lds, int slot, int y, int k0) {
  for (int h = 0; h * kWave < (1 << g.lw) + 2 * g.r; ++h) {
    RowLoads<F, F16, R> in;
    in.load(g, h, y, k0);
    in.store(g, lds, h, slot);
  }
}

// Walks R frames (from the window's k0-th on) of the windows of the wave's pixels.
template <int F, bool F16, int R>
__device__ __forceinline__ void tile_frames(const TileGeom<F, F16>& g, float4* lds, int k0, CellSums<F>& c,
                                            LaneSums<F>& ls) {
  const double K = g.kexp;
  constexpr int NQ = tile_quads(F), U = tile_units(F, R);
  // A wave alone on its SIMD loads the next row while it walks this one; where
  // two share it, the other one walks meanwhile and the registers are short.
  constexpr bool AHEAD = regress_waves_per_simd(F, false) == 1;
  const int r = g.r, TH = kWave >> g.lw, rowpx = (1 << g.lw) + 2 * r;
  wave_lds_order();                                            // after the reads of an earlier walk
  for (int s = 0; s + 1 < TH; ++s) stage_row<F, F16, R>(g, lds, s, g.y0 - r + s, k0);
  const double kxx = K * g.vx_step * g.vx_step;
  const float4* base = lds + static_cast<int>(threadIdx.x & ((1u << g.lw) - 1u)) * U;
  int slot = g.py - g.y0;                                      // of this lane's row
  int next = TH - 1;                                           // of the row to stage
  RowLoads<F, F16, R> in[2];
  if constexpr (AHEAD) {
    in[0].load(g, 0, g.y0 - r + TH - 1, k0);
    in[1].load(g, 1, g.y0 - r + TH - 1, k0);
  }
#pragma unroll 1
  for (int dy = -r; dy <= r; ++dy) {
    if constexpr (AHEAD) {
      in[0].store(g, lds, 0, next);
      in[1].store(g, lds, 1, next);
      in[0].load(g, 0, g.y0 + dy + TH, k0);                    // past the last row: never stored
      in[1].load(g, 1, g.y0 + dy + TH, k0);
    } else {
      stage_row<F, F16, R>(g, lds, next, g.y0 + dy + TH - 1, k0);
    }
    wave_lds_order();
    const double vy = static_cast<double>(dy) * g.vy_step;
    const double ky = static_cast<uint32_t>(g.py + dy) < static_cast<uint32_t>(g.H) ? K * vy * vy : kDropped;
    const float4* at = base + slot * (rowpx * U);
    float4 q[NQ];                                              // the next sample
#pragma unroll
    for (int k = 0; k < NQ; ++k) q[k] = at[k];
#pragma unroll 1
    for (int dx = -r; dx <= r; ++dx) {
      const double e = fma(kxx, static_cast<double>(dx * dx), ky);
      const double cell = static_cast<uint32_t>(g.px + dx) < static_cast<uint32_t>(g.W) ? e : kDropped;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        float ch[4 * NQ];
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
          ch[4 * k] = q[k].x;
          ch[4 * k + 1] = q[k].y;
          ch[4 * k + 2] = q[k].z;
          ch[4 * k + 3] = q[k].w;
        }
        double v[F], s0 = 0, s1 = 0;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          v[f] = fma(static_cast<double>(ch[f]), g.sf[f], -g.xcs[f]);
          if (f & 1) s1 = fma(v[f], v[f], s1);
          else s0 = fma(v[f], v[f], s0);
        }
        const double arg = fma(s0 + s1, K, cell);
        const double w = static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(arg)));
        const double yd = static_cast<double>(ch[F]);
#pragma unroll
        for (int k = 0; k < NQ; ++k) q[k] = at[(i + 1 < R ? (i + 1) * NQ : U) + k];
        c.add(w, yd, v, i == 0);
      }
      at += U;
      c.end_cell(dx);
    }
    ls.end_line(c, vy);
    wave_lds_order();
    next = next + 1 == TH ? 0 : next + 1;
    slot = slot + 1 == TH ? 0 : slot + 1;
  }
}


// Normal equations of one item (or a lane's share of them).
template <int F, class Real = double>
struct Gram {
  static constexpr int NA = F * (F + 1) / 2;
  Real SW, A0y, g0, A0f[F];
  Real A0x, Axx, Axy, gx, Axf[F];
  Real Ayy, gy, Syy, Ayf[F], gf[F], Aff[NA];

  // Calls fn on every total, in a fixed order.
  template <class Fn>
  __device__ __forceinline__ void each(Fn&& fn) {
    fn(SW);
    fn(A0y);
    fn(g0);
    fn(A0x);
    fn(Axx);
    fn(Axy);
    fn(gx);
    fn(Ayy);
    fn(gy);
    fn(Syy);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      fn(A0f[f]);
      fn(Axf[f]);
      fn(Ayf[f]);
      fn(gf[f]);
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) fn(Aff[k]);
  }
  // Applies one DPP butterfly step to every total; the steps run in sequence
  // over all totals (step-major), so consecutive DPP reads never depend on
  // the previous instruction.
  template <int CTRL>
  __device__ __forceinline__ void dpp_step() {
    auto st = [](Real& v) { v += dpp_d<CTRL>(v); };
    st(SW);
    st(A0y);
    st(g0);
    st(A0x);
    st(Axx);
    st(Axy);
    st(gx);
    st(Ayy);
    st(gy);
    st(Syy);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      st(A0f[f]);
      st(Axf[f]);
      st(Ayf[f]);
      st(gf[f]);
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) st(Aff[k]);
  }
  // Over one or two lanes (scatter_sum: more).
  template <int L>
  __device__ __forceinline__ void lane_sum() {
    static_assert(L <= 2);
    if constexpr (L == 2) dpp_step<0xB1>();
  }
};

// Totals of the lane's part of its item from its walk: along columns (v_y is the
// walked coordinate, steps of s, and v_x the lines' one) or, ROWS, along rows.
template <int F, bool ROWS = false>
__device__ __forceinline__ void gram_of_lane(const CellSums<F>& c, const LaneSums<F>& l, double s,
                                             Gram<F, double>& G) {
  G.SW = l.W;
  G.g0 = l.g;
  G.Syy = c.p.Syy;
  G.A0x = ROWS ? s * l.YW : l.XW;
  G.A0y = ROWS ? l.XW : s * l.YW;
  G.Axx = ROWS ? s * s * c.YY : l.XX;
  G.Ayy = ROWS ? l.XX : s * s * c.YY;
  G.gx = ROWS ? s * c.Yg : l.Xg;
  G.gy = ROWS ? l.Xg : s * c.Yg;
  G.Axy = s * l.XY;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    G.A0f[f] = l.f[f];
    G.gf[f] = c.p.gf[f];
    G.Axf[f] = ROWS ? s * c.Yf[f] : l.Xf[f];
    G.Ayf[f] = ROWS ? l.Xf[f] : s * c.Yf[f];
  }
#pragma unroll
  for (int k = 0; k < Gram<F, double>::NA; ++k) G.Aff[k] = c.p.Aff[k];
}

// The moments of one column or part of it; its walk ended at e.
template <int F>
struct ColumnMoments {
  double Y, YY, Yg, Yf[F];
  __device__ __forceinline__ ColumnMoments(const RunSums<F>& c, double e)
      : Y(fma(e, c.W, -c.PW)), YY(fma(e * e, c.W, fma(-(2.0 * e + 1.0), c.PW, 2.0 * c.PPW))), Yg(fma(e, c.g, -c.Pg)) {
#pragma unroll
    for (int f = 0; f < F; ++f) Yf[f] = fma(e, c.f[f], -c.Pf[f]);
  }
  __device__ __forceinline__ ColumnMoments(const CellSums<F>& c, double) : Y(c.YW), YY(c.YY), Yg(c.Yg) {
#pragma unroll
    for (int f = 0; f < F; ++f) Yf[f] = c.Yf[f];
  }
};

// The same for one column or part of it, at v_x.
template <int F, class Sums>
__device__ __forceinline__ void gram_of_column(const Sums& c, double vx, double s, double e, Gram<F, double>& G) {
  const ColumnMoments<F> m(c, e);
  G.SW = c.W;
  G.g0 = c.g;
  G.Syy = c.p.Syy;
  G.A0x = vx * c.W;
  G.Axx = vx * G.A0x;
  G.gx = vx * c.g;
  G.A0y = s * m.Y;
  G.Ayy = s * s * m.YY;
  G.Axy = vx * G.A0y;
  G.gy = s * m.Yg;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    G.A0f[f] = c.f[f];
    G.gf[f] = c.p.gf[f];
    G.Axf[f] = vx * c.f[f];
    G.Ayf[f] = s * m.Yf[f];
  }
#pragma unroll
  for (int k = 0; k < Gram<F, double>::NA; ++k) G.Aff[k] = c.p.Aff[k];
}

// The Gram of the window of the lane's pixel.  The sums of each count of frames
// live and die in their own branch: kept across the branches, the register
// allocator had fitted one of the five walks and spilled 28 to 56 registers at
// every row of the others (640 x 480, F = 7, r = 7: one frame 339 -> 251 us, two 571
// -> 409, three 644 -> 574; F = 8, two frames 2181 -> 573).  The rest, windows of more
// frames than are walked at a time, keeps its sums over a loop of a single walk
// for the same reason (seven frames, r = 5: 919 -> 916 us, F = 10 1811 -> 1726).
template <int F, bool F16>
__device__ __forceinline__ void tile_gram(const TileGeom<F, F16>& g, float4* lds, Gram<F, double>& G) {
  auto whole = [&](auto frames) {
    CellSums<F> c;
    LaneSums<F> ls;
    c.zero();
    ls.zero();
    tile_frames<F, F16, decltype(frames)::value>(g, lds, 0, c, ls);
    gram_of_lane<F, true>(c, ls, g.vx_step, G);
  };
  constexpr int MAX = max_tile_frames(F);
  if (MAX >= 3 && g.nt == 3) whole(std::integral_constant<int, MAX >= 3 ? 3 : 1>{});
  else if (MAX >= 5 && g.nt == 5) whole(std::integral_constant<int, MAX >= 5 ? 5 : 1>{});
  else if (MAX >= 4 && g.nt == 4) whole(std::integral_constant<int, MAX >= 4 ? 4 : 1>{});
  else if (MAX >= 2 && g.nt == 2) whole(std::integral_constant<int, MAX >= 2 ? 2 : 1>{});
  else if (MAX >= 2 && g.nt == 1) whole(std::integral_constant<int, 1>{});
  else {
    CellSums<F> c;
    LaneSums<F> ls;
    c.zero();
    ls.zero();
#pragma unroll 1
    for (int k0 = 0; k0 < g.nt; ++k0) tile_frames<F, F16, 1>(g, lds, k0, c, ls);
    gram_of_lane<F, true>(c, ls, g.vx_step, G);
  }
}

// The Gram of the columns j, j + L, ... of the lane's item, read from memory.  The
// sums of each count of frames have their own branch, as in tile_gram (kept across
// the branches, every row spilled: F = 8, r = 12, five frames, half precision, 307200
// pixels 14.2 ms, now 4.2; the condition output at F = 8, r = 5, 76800 pixels, one
// frame 434 us, now 145).  Frames one at a time with two rows ahead for scattered
// items (lists), whose loads take longer than a cell's samples (20000 items, F = 10,
// r = 7, three frames, one lane: 655 us, three frames at a time 813), for F above 10,
// whose three frames at a time spill, and for more than three frames.
template <int F, int L, bool F16>
__device__ __forceinline__ void walk_gram(const WalkGeom<F, F16>& g, int j, bool dense, Gram<F, double>& G) {
  auto walk = [&](auto frames, auto depth, int chunks) {
    CellSums<F> c;
    LaneSums<F> ls;
    c.zero();
    ls.zero();
#pragma unroll 1
    for (int d0 = -g.r; d0 <= g.r; d0 += L) {
#pragma unroll 1
      for (int k = 0; k < chunks; ++k)
        walk_frames<F, F16, decltype(frames)::value, decltype(depth)::value>(g, d0 + j, k, c);
      ls.end_line(c, static_cast<double>(d0 + j) * g.vx_step);
    }
    gram_of_lane(c, ls, g.vy_step, G);
  };
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  using Three = std::integral_constant<int, 3>;
  constexpr bool CELLS = F < 11;           // two or three frames at a time
  if (CELLS && dense && g.nt == 3) walk(std::conditional_t<CELLS, Three, One>{}, One{}, 1);
  else if (CELLS && dense && g.nt == 2) walk(std::conditional_t<CELLS, Two, One>{}, One{}, 1);
  else walk(One{}, Two{}, g.nt);
}

// ---- lane sums that leave each total in one lane ---------------------------
//
// A step halves both the lanes that share a value and the values a lane holds:
// partners exchange a pair (a, b), one keeps a's sum and the other b's.  The L
// lanes of an item lie in all four rows of 16 lanes (item_slot, item_lane), so
// the first two steps are row swaps: two swaps and an add for each of the 33 and
// 17 pairs at F = 7.  With the two steps inside a quad that is 250 instructions
// for the 66 totals over 16 lanes, where summing every total in every lane takes
// 12 per total.  (Loads do not mind the spread: the vector memory path returns
// eight lanes a cycle whether 64, 16 or 4 neighbouring lanes read one line.)

// Item of the wave (64 / L of them) and lane of the item, from the wave's lane.
template <int L>
__device__ __forceinline__ int item_slot(int lane) { return (lane & 15) / (L / 4); }
template <int L>
__device__ __forceinline__ int item_lane(int lane) { return (lane >> 4) * (L / 4) + (lane & (L / 4 - 1)); }

// Partners in the other half of the wave (ROWS = 2) or in the neighbouring row
// of each half (ROWS = 1): the lower one keeps the sum of a, the upper one b's.
template <int ROWS>
__device__ __forceinline__ double row_sum(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  uint32_t lo[2] = {static_cast<uint32_t>(x), static_cast<uint32_t>(y)};
  uint32_t hi[2] = {static_cast<uint32_t>(x >> 32), static_cast<uint32_t>(y >> 32)};
  if constexpr (ROWS == 2) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo[0], lo[1], false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi[0], hi[1], false, false);
    lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(lo[0], lo[1], false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi[0], hi[1], false, false);
    lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
  }
  return __builtin_bit_cast(double, static_cast<uint64_t>(hi[0]) << 32 | lo[0]) +
         __builtin_bit_cast(double, static_cast<uint64_t>(hi[1]) << 32 | lo[1]);
}

// Partners at lane distance D inside a quad.
template <int D>
__device__ __forceinline__ double quad_sum(double a, double b, int lane) {
  const bool up = (lane & D) != 0;
  const double keep = up ? b : a, send = up ? a : b;
  return keep + dpp_d<D == 2 ? 0x4E : 0xB1>(send);     // quad_perm [2,3,0,1], [1,0,3,2]
}

// Sums s over the L lanes of each item; afterwards value e is register
// total_pos(e) / L of the item's lane total_pos(e) % L.
template <int L, int N, int STEP = 0>
__device__ __forceinline__ void scatter_sum(double (&s)[N], int lane) {
  constexpr int M = (N + 1) / 2;
  double t[M];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const double a = s[2 * k], b = 2 * k + 1 < N ? s[2 * k + 1] : 0.0;
    if constexpr (STEP == 0) t[k] = row_sum<2>(a, b);
    else if constexpr (STEP == 1) t[k] = row_sum<1>(a, b);
    else t[k] = quad_sum<(L >> (STEP + 1))>(a, b, lane);
  }
  if constexpr ((L >> (STEP + 1)) > 1) scatter_sum<L, M, STEP + 1>(t, lane);
#pragma unroll
  for (int k = 0; k < M; ++k) s[k] = t[k];
}

template <int L>
__host__ __device__ constexpr int total_pos(int e) {
  int low = 0;
  for (int b = 1, m = L >> 1; b < L; b <<= 1, m >>= 1)
    if (e & b) low |= m;
  return e / L * L + low;
}

// Walks the lane's part of its item's window (lane j of L) and calls fn(G, first)
// with the totals of each turn, to be summed over the turns: no sums are kept in
// registers from one turn to the next, so that a turn has room for two rows of
// loads ahead.  A turn is up to three frames of a column per lane; where fewer
// than L columns are left (q), each is cut into L / q parts of equal height, one
// lane each, so that the last turn is as short as the lanes allow: at r = 9,
// 16 lanes walk 19 rows of 16 columns and then 4 rows of the last 3 columns (5
// lanes a column).  kListSingle: one turn of uncut columns (L / 2 < 2 r + 1 <= L, at
// most three frames).  With whole columns in every turn, sums kept in registers
// between turns and so one row of loads ahead, lists of 65536 / 4096 items (one in
// eight pixels of a wide image, F = 7, three frames) took 98 / 14 us at r = 3, 392 /
// 39 at r = 8, 426 / 42 at r = 9 and 537 / 50 at r = 12; now 84 / 14, 282 / 29, 324 /
// 30 and 500 / 46.  F = 10, r = 10, five frames: 1344 / 95, now 955 / 69.
template <int F, int L, bool F16, int KIND, class Fn>
__device__ __forceinline__ void walk_parts(const WalkGeom<F, F16>& g, int j, Fn&& fn) {
  // two rows ahead where they fit the registers (two waves per SIMD to F = 8, one
  // above): at F = 8, r = 10, five frames, 18000 items spilled to 303 us, 232 with one
  constexpr int DEPTH = F == 12 || (F == 8 && KIND != kListSingle) ? 1 : 2;
  std::conditional_t<KIND == kListExact, CellSums<F>, RunSums<F>> c;
  Gram<F, double> got;
  if constexpr (KIND == kListSingle) {
    const int dx = j - g.r;
    c.zero();
    if (g.nt == 3) walk_frames<F, F16, 3, DEPTH>(g, dx, 0, c);
    else if (g.nt == 2) walk_frames<F, F16, 2, DEPTH>(g, dx, 0, c);
    else walk_frames<F, F16, 1, DEPTH>(g, dx, 0, c);
    gram_of_column(c, static_cast<double>(dx) * g.vx_step, g.vy_step, static_cast<double>(g.r + 1), got);
    fn(got, true);
  } else {
    const int span = 2 * g.r + 1;
#pragma unroll 1
    for (int d0 = 0; d0 < span; d0 += L) {
      const int q = min(L, span - d0), parts = L / q, n = (span + parts - 1) / parts;
      // idle lanes (part >= parts) and rows past the window walk with weight 0
      const int part = j / q;
      const int dx = part < parts ? d0 + j - part * q - g.r : g.r + 1;
      const int s0 = part * n - g.r;
#pragma unroll 1
      for (int k0 = 0; k0 < g.nt; k0 += 3) {
        const int left = g.nt - k0;
        c.zero();
        if (left >= 3) walk_frames<F, F16, 3, DEPTH, true>(g, dx, k0, c, s0, n);
        else if (left == 2) walk_frames<F, F16, 2, DEPTH, true>(g, dx, k0, c, s0, n);
        else walk_frames<F, F16, 1, DEPTH, true>(g, dx, k0, c, s0, n);
        gram_of_column(c, static_cast<double>(dx) * g.vx_step, g.vy_step, static_cast<double>(s0 + n), got);
        fn(got, d0 == 0 && k0 == 0);
      }
    }
  }
}

// Neumaier-compensated accumulation: (hi, lo) += x.
__device__ __forceinline__ void neumaier(float& hi, float& lo, float x) {
  const float t = hi + x;
  lo += fabsf(hi) >= fabsf(x) ? (hi - t) + x : (x - t) + hi;
  hi = t;
}

// FP32 normal equations with block-compensated sums: every sample updates
// plain FP32 partials of the current column pass (a block of 2tr+1 times
// 2r+1 samples); at the end of the pass each partial is added to a
// Neumaier-compensated (hi, lo) total, and lane groups merge their totals
// with error-free two-sums.  Values are read back as hi + lo.
template <int F>
struct GramC {
  static constexpr int NA = F * (F + 1) / 2;
  static constexpr int NQ = F + 3;             // qW, qY, qG, qF[F]
  static constexpr int ND = 3 + 2 * F + NA;    // Ayy, gy, Syy, Ayf[F], gf[F], Aff[NA]
  static constexpr int NT = 2 * NQ + 1 + ND;   // q totals, x folds, Axx, directs
  float q[NQ], d[ND];
  float hi[NT], lo[NT];

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int k = 0; k < NT; ++k) hi[k] = lo[k] = 0.0f;
  }
  __device__ __forceinline__ void pass_begin() {
#pragma unroll
    for (int k = 0; k < NQ; ++k) q[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < ND; ++k) d[k] = 0.0f;
  }
  __device__ __forceinline__ void add(float w, float yd, const float (&v)[F], float vy) {
    const float wy = w * yd;
    const float wvy = w * vy;
    q[0] += w;
    q[1] += wvy;
    q[2] += wy;
    d[0] = fmaf(wvy, vy, d[0]);
    d[1] = fmaf(wy, vy, d[1]);
    d[2] = fmaf(wy, yd, d[2]);
    int qq = 0;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const float wz = w * v[f];
      q[3 + f] += wz;
      d[3 + f] = fmaf(wvy, v[f], d[3 + f]);
      d[3 + F + f] = fmaf(wz, yd, d[3 + F + f]);
#pragma unroll
      for (int e = f; e < F; ++e) {
        d[3 + 2 * F + qq] = fmaf(wz, v[e], d[3 + 2 * F + qq]);
        ++qq;
      }
    }
  }
  __device__ __forceinline__ void pass_end(float vx) {
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      neumaier(hi[k], lo[k], q[k]);
      neumaier(hi[NQ + k], lo[NQ + k], vx * q[k]);
    }
    neumaier(hi[2 * NQ], lo[2 * NQ], vx * vx * q[0]);
#pragma unroll
    for (int k = 0; k < ND; ++k) neumaier(hi[2 * NQ + 1 + k], lo[2 * NQ + 1 + k], d[k]);
  }
  template <int L>
  __device__ __forceinline__ void lane_sum() {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      float h = hi[k], l = lo[k];
      auto step = [&](float h2, float l2) {
        const float s = h + h2;
        const float bb = s - h;
        const float err = (h - (s - bb)) + (h2 - bb);
        h = s;
        l = l + l2 + err;
      };
      if constexpr (L >= 2) step(dpp_f<0xB1>(h), dpp_f<0xB1>(l));
      if constexpr (L >= 4) step(dpp_f<0x4E>(h), dpp_f<0x4E>(l));
      if constexpr (L >= 8) step(dpp_f<0x141>(h), dpp_f<0x141>(l));
      if constexpr (L >= 16) step(dpp_f<0x140>(h), dpp_f<0x140>(l));
      hi[k] = h;
      lo[k] = l;
    }
  }
  // Totals in the Gram layout, as Real (hi + lo evaluated in Real).
  template <class Real>
  __device__ __forceinline__ void values(Gram<F, Real>& G) const {
    auto v = [&](int k) { return static_cast<Real>(hi[k]) + static_cast<Real>(lo[k]); };
    G.SW = v(0);
    G.A0y = v(1);
    G.g0 = v(2);
    G.A0x = v(NQ + 0);
    G.Axy = v(NQ + 1);
    G.gx = v(NQ + 2);
    G.Axx = v(2 * NQ);
    G.Ayy = v(2 * NQ + 1);
    G.gy = v(2 * NQ + 2);
    G.Syy = v(2 * NQ + 3);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      G.A0f[f] = v(3 + f);
      G.Axf[f] = v(NQ + 3 + f);
      G.Ayf[f] = v(2 * NQ + 4 + f);
      G.gf[f] = v(2 * NQ + 4 + F + f);
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) G.Aff[k] = v(2 * NQ + 4 + 2 * F + k);
  }
};

__host__ __device__ constexpr int tri(int i, int j) { return i * (i + 1) / 2 + j; }

// Wave-group iteration with XCD affinity.  Workgroups are dispatched to the
// nxcd XCDs round-robin by block index, so block b runs on XCD b % nxcd.  When
// the grid is a multiple of nxcd blocks, XCD x walks a contiguous range of the
// groups (the x-th of nxcd equal parts, or [xb[x], xb[x + 1]) when a split by
// work is given), which keeps spatially adjacent items (sharing window rows)
// in the same L2; otherwise a plain grid stride is used.
struct GroupIter {
  int64_t g, end, step;
  __device__ __forceinline__ GroupIter(int64_t ngroups, int nxcd, const int64_t* xb = nullptr) {
    const int64_t nblk = gridDim.x;
    const int64_t wib = uni(static_cast<int>(threadIdx.x) / kWave);   // wave in block
    const int64_t wpb = blockDim.x / kWave;
    const int64_t nx = nxcd;
    if (nx > 1 && nblk >= nx && nblk % nx == 0) {
      const int64_t x = blockIdx.x % nx;
      int64_t lo, hi;
      if (xb) {
        lo = xb[x];
        hi = min(ngroups, xb[x + 1]);
      } else {
        const int64_t chunk = (ngroups + nx - 1) / nx;
        lo = x * chunk;
        hi = min(ngroups, (x + 1) * chunk);
      }
      g = lo + (blockIdx.x / nx) * wpb + wib;
      end = hi;
      step = (nblk / nx) * wpb;
    } else {
      g = static_cast<int64_t>(blockIdx.x) * wpb + wib;
      end = ngroups;
      step = nblk * wpb;
    }
  }
  __device__ __forceinline__ bool next(int64_t& out) {
    if (g >= end) return false;
    out = g;
    g += step;
    return true;
  }
};

// The groups of a launch of one block per CU: each block gets an equal share and
// its waves fetch one after the other from a counter in LDS, so that a wave that
// is issued less often (or that waits longer for memory) gets fewer.  Which wave
// runs a group does not matter to its results.  One clip: a share is a run of
// consecutive groups (neighbouring pixels in the CU's L1), the XCDs' blocks side
// by side.  Several clips, whose groups cost in proportion to their windows:
// every nblk-th group.
struct GroupQueue {
  int64_t first, step, count;      // the block's groups: first + k step, k < count
  int* taken;                      // LDS: groups handed out

  __device__ __forceinline__ GroupQueue(int64_t ngroups, int nclips, int nxcd, int* counter) : taken(counter) {
    const int64_t nblk = gridDim.x, nx = nblk % nxcd == 0 ? nxcd : 1;
    const int64_t b = static_cast<int64_t>(blockIdx.x % nx) * (nblk / nx) + blockIdx.x / nx;
    first = nclips == 1 ? b * ngroups / nblk : b;
    step = nclips == 1 ? 1 : nblk;
    count = nclips == 1 ? (b + 1) * ngroups / nblk - first : ngroups > b ? (ngroups - b + nblk - 1) / nblk : 0;
    if (threadIdx.x == 0) *taken = static_cast<int>(blockDim.x / kWave);
    __syncthreads();
  }
  // The wave's first group, as its index k in the block's share: waves side by
  // side lie on different SIMDs, so that a share of a few groups spreads over them.
  __device__ __forceinline__ int64_t start() const { return uni(static_cast<int>(threadIdx.x) / kWave); }
  // The wave's next group (uniform over the wave); from `count` on there is none.
  __device__ __forceinline__ int64_t next() const {
    int k = 0;
    if ((threadIdx.x & (kWave - 1)) == 0) k = atomicAdd(taken, 1);
    return uni(k);
  }
  __device__ __forceinline__ int64_t group(int64_t k) const { return first + k * step; }
};

// Hardware estimates of 1/sqrt(x) and 1/x.
__device__ __forceinline__ double rsq_approx(double x) { return __builtin_amdgcn_rsq(x); }
__device__ __forceinline__ float rsq_approx(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rcp_approx(double x) { return __builtin_amdgcn_rcp(x); }
__device__ __forceinline__ float rcp_approx(float x) { return __builtin_amdgcn_rcpf(x); }

// 1/sqrt(x) refined by two Newton steps from the hardware estimate (each step
// doubles the correct bits; within an ulp or two of the correctly rounded
// value, a short dependent chain instead of the correctly rounded square root
// and divide sequences).
template <class Real>
__device__ __forceinline__ Real rsq_refined(Real x) {
  Real y = rsq_approx(x);
  y = y * fma(Real(-0.5) * x * y, y, Real(1.5));
  y = y * fma(Real(-0.5) * x * y, y, Real(1.5));
  return y;
}

// Solves L L^T x = b with the packed factor (its diagonal holds 1 / L_ii).
template <int P, class Real>
__device__ __forceinline__ void chol_solve(const Real (&M)[P * (P + 1) / 2], const Real (&b)[P],
                                           Real (&x)[P]) {
#pragma unroll
  for (int i = 0; i < P; ++i) {
    Real v = b[i];
#pragma unroll
    for (int k = 0; k < i; ++k) v -= M[tri(i, k)] * x[k];
    x[i] = v * M[tri(i, i)];
  }
#pragma unroll
  for (int i = P - 1; i >= 0; --i) {
    Real v = x[i];
#pragma unroll
    for (int k = i + 1; k < P; ++k) v -= M[tri(k, i)] * x[k];
    x[i] = v * M[tri(i, i)];
  }
}

// In-place packed Cholesky A = L L^T; the diagonal slots receive 1 / L_ii (the
// solves multiply by it), from the refined reciprocal square root of the
// pivot.  A non-positive pivot yields NaN.
template <int P, class Real>
__device__ __forceinline__ void cholesky_inplace(Real (&M)[P * (P + 1) / 2]) {
#pragma unroll
  for (int c = 0; c < P; ++c) {
    Real s = M[tri(c, c)];
#pragma unroll
    for (int k = 0; k < c; ++k) s -= M[tri(c, k)] * M[tri(c, k)];
    Real id = rsq_refined(s);
    id = s > Real(0) ? id : static_cast<Real>(__builtin_nan(""));
    M[tri(c, c)] = id;
#pragma unroll
    for (int i = c + 1; i < P; ++i) {
      Real v = M[tri(i, c)];
#pragma unroll
      for (int k = 0; k < c; ++k) v -= M[tri(i, k)] * M[tri(c, k)];
      M[tri(i, c)] = v * id;
    }
  }
}

// Assembles the W-normalised system in scaled units (unknowns alpha, beta_x,
// beta_y, beta_f..), adds the scaled ridge, factors it in place (packed lower
// Cholesky) and solves for theta.  Returns 1/W.  anorm1 receives the 1-norm of
// the equilibrated matrix S^-1 A S^-1 (S^2 = diag(A), unit diagonal), for the
// condition estimate (equilibrate_factor, hager_inv_norm1).
template <int F, class Real>
__device__ __forceinline__ Real gram_solve(const Gram<F, Real>& G, const ClipDev& C,
                                           Real (&M)[(F + 3) * (F + 4) / 2], Real (&rhs)[F + 3],
                                           Real (&th)[F + 3], Real& anorm1) {
  constexpr int P = F + 3;
  const Real iW = Real(1) / G.SW;
  const Real lam = static_cast<Real>(C.ridge);
  M[tri(0, 0)] = Real(1);
  M[tri(1, 0)] = G.A0x * iW;
  M[tri(2, 0)] = G.A0y * iW;
  M[tri(1, 1)] = G.Axx * iW + lam * static_cast<Real>(C.c2[0]);
  M[tri(2, 1)] = G.Axy * iW;
  M[tri(2, 2)] = G.Ayy * iW + lam * static_cast<Real>(C.c2[1]);
  rhs[0] = G.g0 * iW;
  rhs[1] = G.gx * iW;
  rhs[2] = G.gy * iW;
  {
    int q = 0;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      M[tri(3 + f, 0)] = G.A0f[f] * iW;
      M[tri(3 + f, 1)] = G.Axf[f] * iW;
      M[tri(3 + f, 2)] = G.Ayf[f] * iW;
      rhs[3 + f] = G.gf[f] * iW;
#pragma unroll
      for (int e = f; e < F; ++e) {
        M[tri(3 + e, 3 + f)] = G.Aff[q] * iW + (e == f ? lam * static_cast<Real>(C.c2[2 + f]) : Real(0));
        ++q;
      }
    }
  }
  Real isd[P];
#pragma unroll
  for (int i = 0; i < P; ++i) isd[i] = Real(1) / sqrt(M[tri(i, i)]);
  anorm1 = 0;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    Real cs = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) cs += fabs(i >= c ? M[tri(i, c)] : M[tri(c, i)]) * isd[i];
    anorm1 = fmax(anorm1, cs * isd[c]);
  }
  cholesky_inplace<P, Real>(M);
  chol_solve<P, Real>(M, rhs, th);
  return iW;
}


// Turns the packed Cholesky factor of A (diagonal slots holding 1 / L_ii) into
// the factor of the equilibrated As = S^-1 A S^-1, S^2 = diag(A): row i of L
// divided by S_i, with A_ii = sum_k L_ik^2 read off the factor itself.  In
// place; M is no longer A's factor afterwards.  By van der Sluis the rounding
// error of the Cholesky solve is governed by kappa(As), not kappa(A), whose
// diagonal spans the ridge (a constant feature) to 1.
template <int P, class Real>
__device__ __forceinline__ void equilibrate_factor(Real (&M)[P * (P + 1) / 2]) {
#pragma unroll
  for (int i = 0; i < P; ++i) {
    // A_ii = L_ii^2 + sum_k L_ik^2, with L_ii = 1 / M_ii (the slot's value)
    const Real lii = rcp_approx(M[tri(i, i)]);
    Real s = lii * lii;
#pragma unroll
    for (int k = 0; k < i; ++k) s += M[tri(i, k)] * M[tri(i, k)];
    // an estimate needs no correctly rounded root: the hardware reciprocal
    // square root (about 1 ulp) keeps this short
    const Real isd = rsq_approx(s), sd = s * isd;
#pragma unroll
    for (int k = 0; k < i; ++k) M[tri(i, k)] *= isd;
    M[tri(i, i)] *= sd;
  }
}

// Estimate of ||A^{-1}||_1 for a symmetric positive definite A from its
// packed Cholesky factor, after Hager (1984) with Higham's refinements (1988,
// the scheme of LAPACK's xLACN2): power-like steps on sign vectors, at most
// five solves with unit vectors, then an extra test vector with alternating
// signs.  kappa_1 is estimated as ||A||_1 times this; the estimate never
// exceeds the true value.
template <int P, class Real>
__device__ __forceinline__ Real hager_inv_norm1(const Real (&M)[P * (P + 1) / 2]) {
  Real b[P], x[P], z[P], xi[P];
  auto norm1 = [&](const Real (&v)[P]) {
    Real s = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) s += fabs(v[i]);
    return s;
  };
  auto argmax_abs = [&](const Real (&v)[P]) {
    int jm = 0;
    Real m = fabs(v[0]);
#pragma unroll
    for (int i = 1; i < P; ++i)
      if (fabs(v[i]) > m) {
        m = fabs(v[i]);
        jm = i;
      }
    return jm;
  };
#pragma unroll
  for (int i = 0; i < P; ++i) b[i] = Real(1) / P;
  chol_solve<P, Real>(M, b, x);
  Real est = norm1(x);
#pragma unroll
  for (int i = 0; i < P; ++i) xi[i] = x[i] >= Real(0) ? Real(1) : Real(-1);
  chol_solve<P, Real>(M, xi, z);
  int j = argmax_abs(z);
#pragma unroll 1
  for (int iter = 0; iter < 4; ++iter) {
#pragma unroll
    for (int i = 0; i < P; ++i) b[i] = i == j ? Real(1) : Real(0);
    chol_solve<P, Real>(M, b, x);
    const Real old = est;
    est = fmax(est, norm1(x));
    bool same = true;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const Real sgn = x[i] >= Real(0) ? Real(1) : Real(-1);
      same = same && sgn == xi[i];
      xi[i] = sgn;
    }
    if (same || !(est > old)) break;
    chol_solve<P, Real>(M, xi, z);
    const int jn = argmax_abs(z);
    if (fabs(z[jn]) == fabs(z[j])) break;
    j = jn;
  }
  // alternating-sign test vector
#pragma unroll
  for (int i = 0; i < P; ++i)
    b[i] = (i & 1 ? Real(-1) : Real(1)) * (Real(1) + static_cast<Real>(i) / static_cast<Real>(P > 1 ? P - 1 : 1));
  chol_solve<P, Real>(M, b, x);
  est = fmax(est, Real(2) * norm1(x) / (Real(3) * P));
  return est;
}

}  // namespace esim
