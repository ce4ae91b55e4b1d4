// Instantiates the regression, bandwidth and adjoint kernels of one feature count (ESIM_REGRESS_F,
// set by the build) and fills its dispatch table.
#include "esim_backward_impl.h"
#include "esim_bandwidth_impl.h"
#include "esim_regress_impl.h"

#ifndef ESIM_REGRESS_F
#error "ESIM_REGRESS_F must be defined"
#endif

#define ESIM_CAT2(a, b) a##b
#define ESIM_CAT(a, b) ESIM_CAT2(a, b)

namespace esim {

// The instances of 16 lanes per item of one ListKind.
template <int F, int KIND>
void list_kernels(RegressTable& t) {
  t.list[KIND][0] = regress_list_kernel<F, 16, false, KIND>;
  t.list[KIND][1] = regress_list_kernel<F, 16, true, KIND>;
  t.bandwidth_list[KIND][0] = bandwidth_list_kernel<F, false, KIND>;
  t.bandwidth_list[KIND][1] = bandwidth_list_kernel<F, true, KIND>;
  t.adjoint[KIND][0] = adjoint_kernel<F, 16, false, KIND>;
  t.adjoint[KIND][1] = adjoint_kernel<F, 16, true, KIND>;
}

void ESIM_CAT(regress_table_, ESIM_REGRESS_F)(RegressTable& t) {
  constexpr int F = ESIM_REGRESS_F;
  t.lanes1_2[0][0] = regress_kernel<F, 1, false, false>;
  t.lanes1_2[0][1] = regress_kernel<F, 1, true, false>;
  t.lanes1_2[1][0] = regress_kernel<F, 2, false, false>;
  t.lanes1_2[1][1] = regress_kernel<F, 2, true, false>;
  t.lanes4_8[0][0][0] = regress_list_kernel<F, 4, false, kListParts>;
  t.lanes4_8[0][0][1] = regress_list_kernel<F, 4, true, kListParts>;
  t.lanes4_8[0][1][0] = regress_list_kernel<F, 4, false, kListExact>;
  t.lanes4_8[0][1][1] = regress_list_kernel<F, 4, true, kListExact>;
  t.lanes4_8[1][0][0] = regress_list_kernel<F, 8, false, kListParts>;
  t.lanes4_8[1][0][1] = regress_list_kernel<F, 8, true, kListParts>;
  t.lanes4_8[1][1][0] = regress_list_kernel<F, 8, false, kListExact>;
  t.lanes4_8[1][1][1] = regress_list_kernel<F, 8, true, kListExact>;
  list_kernels<F, kListParts>(t);
  list_kernels<F, kListSingle>(t);
  list_kernels<F, kListExact>(t);
  t.tile[0] = regress_tile_kernel<F, false>;
  t.tile[1] = regress_tile_kernel<F, true>;
  t.bandwidth[0][0] = bandwidth_tile_kernel<F, false>;
  t.bandwidth[0][1] = bandwidth_tile_kernel<F, true>;
  t.bandwidth[1][0] = bandwidth_dense_kernel<F, false>;
  t.bandwidth[1][1] = bandwidth_dense_kernel<F, true>;
  t.kappa[0] = regress_kernel<F, 1, false, false, true>;
  t.kappa[1] = regress_kernel<F, 1, true, false, true>;
  // the compensated-FP32 variant is compiled for the feature counts of the
  // workloads (7 and 10) and for the default lane counts
#if ESIM_REGRESS_F == 7 || ESIM_REGRESS_F == 10
  t.c32[0][0] = regress_kernel<F, 4, false, true>;
  t.c32[0][1] = regress_kernel<F, 4, true, true>;
  t.c32[1][0] = regress_kernel<F, 16, false, true>;
  t.c32[1][1] = regress_kernel<F, 16, true, true>;
#endif
}

}  // namespace esim
