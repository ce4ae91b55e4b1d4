// Device buffers of the adjoint (esim_backward.hip) and the item kernel's arguments.
#pragma once

#include "esim_internal.h"

namespace esim {

// Doubles of an item's record: c = g_alpha v / W and theta (F + 3 each),
// q = g_alpha v^T Lambda theta / W, and the scaled centre features.
constexpr int adjoint_record(int F) { return 2 * (F + 3) + 1 + F; }

struct BwdDev {
  int32_t* item_map;   // [T*HW]
  double* rec;         // [n][adjoint_record] per-item records
  double* gbpart;      // [npart][D] per-gather-block bandwidth partials
  double* gbblk;       // [kRedBlocks][D]
  int64_t n;
  int64_t npart;
};

struct AdjointArgs {
  RegressArgs reg;        // single clip: the items, frames from the items
  const float* g_alpha;   // [n] upstream gradients; items with 0 are skipped
  BwdDev bd;
};

}  // namespace esim
