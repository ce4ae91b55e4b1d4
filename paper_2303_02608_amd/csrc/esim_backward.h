// Device buffers of the adjoint (esim_backward.hip) and the item kernel's arguments.
#pragma once

#include "esim_internal.h"

namespace esim {

struct BwdDev {
  int32_t* item_map;   // [T*HW]
  double* rec;         // [n][2P + 1] per-item records (c, theta, q)
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
