// Bandwidth-optimised regression (Sec. 3, bandwidth optimisation): the global
// bandwidth h of eq. (5) chosen per regression from K candidates by the
// smallest estimated mean squared error of alpha.
//
// alpha_h = e_0^T A_h^{-1} g_h is linear in the observations y, and its weight
// on the centre sample (w_c = 1, z_c = e_0) is v_0 / W_h with v = A_h^{-1} e_0.
// With sigma_c^2 the MC variance of y_c, Stein's unbiased risk estimate
//     SURE(h) = (alpha_h - y_c)^2 + 2 sigma_c^2 v_0 / W_h - sigma_c^2
// estimates E[(alpha_h - f_c)^2] (squared bias plus variance).
//
//   log_variance_kernel  sigma^2 of y = log(E + eps) from the radiance sample
//                        variance: var / spp / (E + eps)^2 (delta method).
//   bandwidth_*_kernel   (esim_bandwidth_impl.h) per regression and candidate:
//                        the window walk of the regression with the weights of
//                        that h, Cholesky, theta and v; the outputs of the
//                        candidate with the smallest SURE (the first of equal
//                        ones) are written.
#include <cstdint>

#include "esim_bandwidth.h"
#include "esim_internal.h"

namespace esim {
namespace {

__global__ void __launch_bounds__(256)
log_variance_kernel(const float* __restrict__ E, const float* __restrict__ var, float* __restrict__ vy,
                    int64_t n, float inv_spp, float eps) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const float e = E[i] + eps;
    vy[i] = var[i] * inv_spp / (e * e);
  }
}

}  // namespace

hipError_t launch_log_variance(const float* E, const float* var, float* vy, int64_t n, int spp, float eps,
                               hipStream_t s) {
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(log_variance_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, E, var, vy, n,
                     1.0f / static_cast<float>(spp), eps);
  return hipGetLastError();
}

hipError_t launch_bandwidth(const BandwidthArgs& b, int F, bool f16, int lanes, const DeviceShape& dev, hipStream_t s) {
  const RegressArgs& a = b.reg;
  const RegressTable* t = regress_table(F);
  const BandwidthFn k = !t            ? nullptr
                        : lanes == 16 ? t->bandwidth_list[a.kind][f16]
                                      : t->bandwidth[a.tile_units ? 0 : 1][f16];
  if (!k) return hipErrorInvalidValue;
  return launch_groups(reinterpret_cast<const void*>(k), const_cast<BandwidthArgs*>(&b), a, F,
                       lanes == 16 || a.tile_units, regress_waves_per_simd(F, false), dev, s);
}

}  // namespace esim
