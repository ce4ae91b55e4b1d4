// Which kernel instance runs a clip's FP64 regressions, and how a launch over
// several clips is put together.  Plain host code, no HIP.
//
// An instance fixes the order of a regression's sums.  What a clip gets follows
// from its own shape and parameters (and the schedule, where one was set), never
// from the other clips of its plan: converted in a batch it gives the bits that it
// gives alone.  A launch takes the clips of one instance; a plan of several kinds
// of clips takes one launch for each.
#pragma once

#include <cstddef>
#include <cstdint>

namespace esim {

constexpr int kWave = 64;

// FP64 instances up to 8 features keep their sums within half the register file
// and run two waves per SIMD (a wave's scalar and memory instructions then issue
// beside the other wave's FMAs); larger F, and the compensated-FP32 variant, run
// one.
constexpr int regress_waves_per_simd(int F, bool c32) { return (!c32 && F <= 8) ? 2 : 1; }

constexpr int lanes_index(int L) { return L == 1 ? 0 : L == 2 ? 1 : L == 4 ? 2 : L == 8 ? 3 : 4; }

// Tiles of a dense launch with one lane per pixel (esim_wlr.h): 64 pixels of 2^lw
// columns, each wave with its own LDS.
constexpr int tile_quads(int F) { return (F + 4) / 4; }                            // 16-byte units of F + 1 channels
constexpr int tile_units(int F, int frames) { return (frames * tile_quads(F)) | 1; }   // of a pixel's record
// Frames walked at a time (windows of more: one by one): five, where the rows
// loaded ahead leave the registers for them (F = 12, three frames, 307200 pixels,
// r = 7: spilling with three at a time 3.17 ms, one by one 2.17).
constexpr int max_tile_frames(int F) { return F > 11 ? 1 : F > 10 ? 3 : 5; }
// 16-byte units of a wave's LDS for windows of radius r (the ring of rows), and
// of the record behind a block's last wave that the look-ahead of a row's walk
// may read (of the longest windows: plans mix them).
constexpr int tile_last_units(int F) { return tile_units(F, max_tile_frames(F)); }
constexpr int tile_wave_units(int F, int r, int tr, int lw) {
  return tile_units(F, 2 * tr + 1 < max_tile_frames(F) ? 2 * tr + 1 : max_tile_frames(F)) * ((1 << lw) + 2 * r) *
         (kWave >> lw);
}
constexpr size_t kMaxTileLds = 160 * 1024 - 64;      // of a block (one per CU): the CU's LDS less the queue
constexpr size_t tile_block_bytes(int F, int wave_units) {
  return (static_cast<size_t>(wave_units) * 4u * regress_waves_per_simd(F, false) + tile_last_units(F)) * 16u;
}
constexpr int64_t tile_count(int W, int H, int lw) {
  return static_cast<int64_t>((W + (1ll << lw) - 1) >> lw) * ((H + (kWave >> lw) - 1) / (kWave >> lw));
}

// How the 16-lane instances walk a clip's windows and sum their moments (walk_parts,
// RunSums, CellSums).
enum ListKind { kListParts = 0, kListSingle, kListExact, kListKinds };
// Ridges below this take the instance with exact moments: down to here the others'
// error is at most 4e-9 of the ridge.
constexpr double kExactRidge = 1e-7;

struct ClipRoute {
  int tile_lw;        // log2 of the tiles' width
  bool tiles;         // dense tiles run from LDS
  bool few;           // a dense frame takes 16 lanes per item
  int kind;           // ListKind
};

inline ClipRoute clip_route(int W, int H, int F, int r, int tr, double ridge, int cus) {
  ClipRoute c{};
  // tiles of 64, 32 or 16 columns: of those whose rows are loaded in at most two
  // turns of a wave's lanes and whose ring fits LDS, the one that covers the image
  // with the fewest pixels (the widest of equal ones)
  auto fits = [&](int lw) {
    return (1 << lw) + 2 * r <= 2 * kWave && tile_block_bytes(F, tile_wave_units(F, r, tr, lw)) <= kMaxTileLds;
  };
  c.tile_lw = 6;
  c.tiles = false;
  for (int lw = 6; lw >= 4; --lw)
    if (fits(lw) && (!c.tiles || tile_count(W, H, lw) < tile_count(W, H, c.tile_lw))) {
      c.tile_lw = lw;
      c.tiles = true;
    }
  // A tile is a wave of 64 pixels whatever it covers.  On images narrower than about
  // a tile's smallest width, packed lanes that read from memory do less: 131072 pixels,
  // F = 7, r = 7, three frames: 4 columns 0.87 ms in tiles, 0.28 from memory; 8 columns
  // 0.44 and 0.30; 20 columns, a cover of 0.62, 0.45 and 0.47.
  c.tiles = c.tiles && 5 * static_cast<int64_t>(W) * H >= 3 * kWave * tile_count(W, H, c.tile_lw);
  // A frame of fewer tiles than the device has SIMDs takes as long as one wave over
  // its windows; 16 lanes per item take less up to a share of a tile per SIMD that
  // grows with the window, whose solve the 16 lanes cost extra.  The tiles' time is
  // reached at, of 65536 pixels (256 CUs), one frame or three: r = 1 0.14, r = 2
  // 0.2-0.3, r = 3 0.3-0.4, r = 4 0.4, r = 5 0.5-0.55, r = 6 to 12 0.6-0.8 (F = 1 to
  // 8, 12); F = 9 to 11, whose tiles load rows ahead: r = 3 0.25-0.3, r = 5 0.35-0.4,
  // r = 6 and more 0.4-0.6.  (F = 7, r = 7, three frames: 4096 pixels 129 us in tiles,
  // 18 on 16 lanes; 50176 pixels 131 and 135.  r = 3: 21 and 48 at 57600.)  Where
  // windows are read from memory, 16 lanes are ahead up to a pixel per lane (F = 7,
  // r = 33: 62500 pixels 1.30 and 1.00 ms).
  const int64_t simds = 4ll * cus;
  const int share = r < 6 ? r : 6;
  c.few = c.tiles ? (F >= 9 && F <= 11 ? 14 : 10) * tile_count(W, H, c.tile_lw) < share * simds
                  : static_cast<int64_t>(W) * H < kWave * simds;
  // 9 to 15 columns are one uncut turn of 16 lanes; narrower windows fill the lanes
  // better cut into parts (65536 items at r = 3: 84 us, uncut 98)
  c.kind = ridge < kExactRidge ? kListExact : r >= 4 && r <= 7 && tr <= 1 ? kListSingle : kListParts;
  return c;
}

// Dense launches: the clips that one takes, and their instance.  Of the automatic
// schedule: kDenseFew and the ones after it.
enum DenseSet {
  kDenseLanes = 0,        // + lanes_index(L): every clip, L lanes per item
  kDenseTile = 5,         // one lane per item set by hand: clips whose tiles fit
  kDenseMemory,           //   the others, windows from memory
  kDense16,               // + ListKind: 16 lanes set by hand
  kDenseFew = kDense16 + kListKinds,         // + ListKind: few, 16 lanes
  kDenseAutoTile = kDenseFew + kListKinds,   // not few: tiles, or from memory
  kDenseAutoMemory,
  kDenseSets
};

inline bool dense_member(int set, const ClipRoute& c) {
  if (set < kDenseTile) return true;
  if (set >= kDense16 && set < kDenseFew) return c.kind == set - kDense16;
  if (set >= kDenseFew && set < kDenseAutoTile) return c.few && c.kind == set - kDenseFew;
  const bool tiles = set == kDenseTile || set == kDenseAutoTile;
  return c.tiles == tiles && !(set >= kDenseAutoTile && c.few);
}

constexpr bool dense_tiles(int set) { return set == kDenseTile || set == kDenseAutoTile; }
constexpr int dense_set_lanes(int set) {
  return set < kDenseTile ? 1 << set : set >= kDense16 && set < kDenseAutoTile ? 16 : 1;
}
// ListKind of a set's instance (4 or 8 lanes per item by hand take every clip: exact).
constexpr int dense_kind(int set) {
  return set >= kDenseFew && set < kDenseAutoTile ? set - kDenseFew
         : set >= kDense16 && set < kDenseFew     ? set - kDense16
                                                  : static_cast<int>(kListExact);
}

// Sets that may run kernels whose blocks stride over the groups, XCD by XCD (1, 2, and
// with the compensated Gram 4 and 16 lanes); the others hand their groups out.
constexpr bool dense_strides(int set) {
  return set < kDenseTile ? set != lanes_index(8) : dense_set_lanes(set) == 1 && !dense_tiles(set);
}

// Groups of a clip's pixels in a dense launch: tiles, or 64 / L pixels.
inline int64_t dense_groups(int set, const ClipRoute& c, int W, int H) {
  if (!dense_member(set, c)) return 0;
  if (dense_tiles(set)) return tile_count(W, H, c.tile_lw);
  const int64_t G = kWave / dense_set_lanes(set);
  return (static_cast<int64_t>(W) * H + G - 1) / G;
}

}  // namespace esim
