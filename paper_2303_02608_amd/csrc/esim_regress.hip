// Dispatch of the regression kernels (templates in esim_regress_impl.h, one
// translation unit per feature count).
#include <algorithm>
#include <mutex>

#include "esim_internal.h"

namespace esim {

void regress_table_1(RegressTable&);
void regress_table_2(RegressTable&);
void regress_table_3(RegressTable&);
void regress_table_4(RegressTable&);
void regress_table_5(RegressTable&);
void regress_table_6(RegressTable&);
void regress_table_7(RegressTable&);
void regress_table_8(RegressTable&);
void regress_table_9(RegressTable&);
void regress_table_10(RegressTable&);
void regress_table_11(RegressTable&);
void regress_table_12(RegressTable&);

namespace {

const RegressTable* make_table(int F) {
  static RegressTable tabs[ESIM_MAX_F + 1];
  static std::once_flag once;
  std::call_once(once, [] {
    void (*fill[ESIM_MAX_F + 1])(RegressTable&) = {
        nullptr,          regress_table_1, regress_table_2,  regress_table_3, regress_table_4,
        regress_table_5,  regress_table_6, regress_table_7,  regress_table_8, regress_table_9,
        regress_table_10, regress_table_11, regress_table_12};
    for (int f = 1; f <= ESIM_MAX_F; ++f) fill[f](tabs[f]);
  });
  return (F >= 1 && F <= ESIM_MAX_F) ? &tabs[F] : nullptr;
}

}  // namespace

const RegressTable* regress_table(int F) { return make_table(F); }

namespace {

KernelFn pick(int F, int lanes, int kind, bool f16) {
  const RegressTable* t = regress_table(F);
  if (!t) return nullptr;
  switch (lanes) {
    case 1:
    case 2: return t->lanes1_2[lanes - 1][f16];
    case 4:
    case 8: return t->lanes4_8[lanes == 8][kind == kListExact][f16];
    case 16: return t->list[kind][f16];
    default: return nullptr;
  }
}

KernelFn pick_c32(int F, int lanes, bool f16) {
  const RegressTable* t = regress_table(F);
  const int li = lanes == 4 ? 0 : lanes == 16 ? 1 : -1;
  return (t && li >= 0) ? t->c32[li][f16] : nullptr;
}

}  // namespace

bool regress_supports(int F, int lanes, int precision) {
  if (precision == ESIM_GRAM_F32C) return pick_c32(F, lanes, false) != nullptr;
  return pick(F, lanes, kListParts, false) != nullptr;
}

hipError_t launch_regress(const RegressArgs& a, int F, bool f16, int precision, int lanes,
                          int blocks_per_cu, const DeviceShape& dev, hipStream_t s) {
  // the condition estimate (FP64 Gram) has an instance of its own, one lane
  // per item (the caller sizes the groups for one lane)
  const RegressTable* tab = regress_table(F);
  const bool c32 = precision == ESIM_GRAM_F32C;
  KernelFn fn = c32          ? pick_c32(F, lanes, f16)
                : a.kappa    ? (tab ? tab->kappa[f16] : nullptr)
                : a.tile_units ? (tab ? tab->tile[f16] : nullptr)
                             : pick(F, lanes, a.kind, f16);
  if (!fn) return hipErrorInvalidValue;
  // Tiles and the instances of 4 lanes and more hand out their groups themselves;
  // the others stride over them with the resident blocks (more would only start
  // when those end).
  const int resident = regress_waves_per_simd(F, c32);
  return launch_groups(reinterpret_cast<const void*>(fn), const_cast<RegressArgs*>(&a), a, F,
                       a.tile_units || (!c32 && !a.kappa && lanes >= 4), std::min(blocks_per_cu, resident), dev, s);
}

hipError_t allow_tile_lds(int F, bool f16) {
  const RegressTable* t = regress_table(F);
  if (!t) return hipErrorInvalidValue;
  for (const void* fn : {reinterpret_cast<const void*>(t->tile[f16]), reinterpret_cast<const void*>(t->bandwidth[0][f16])}) {
    const hipError_t e =
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMaxTileLds));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_groups(const void* fn, void* args, const RegressArgs& a, int F, bool queue,
                         int blocks_per_cu, const DeviceShape& dev, hipStream_t s) {
  const int waves = queue ? 4 * regress_waves_per_simd(F, false) : kWavesPerBlock;
  int64_t blocks = queue ? a.max_groups : (a.max_groups + waves - 1) / waves;
  const int64_t cap = static_cast<int64_t>(dev.cus) * (queue ? 1 : blocks_per_cu);
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  blocks = (blocks + dev.xcds - 1) / dev.xcds * dev.xcds;   // a multiple of the XCDs (see GroupIter, GroupQueue)
  const size_t lds = a.tile_units ? tile_block_bytes(F, a.tile_units) : 0;   // allow_tile_lds allows it
  void* argv[] = {args};
  const hipError_t e = hipLaunchKernel(fn, dim3(static_cast<unsigned>(blocks)),
                                       dim3(static_cast<unsigned>(kWave * waves)), argv, lds, s);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace esim
