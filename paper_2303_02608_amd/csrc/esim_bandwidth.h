// Launchers of the bandwidth-optimised regression (esim_bandwidth.hip).
#pragma once

#include "esim_internal.h"

namespace esim {

constexpr int kMaxBandwidths = 8;

struct BandwidthArgs {
  RegressArgs reg;              // single clip: items (nullptr = every pixel), count, frame, alpha, beta
  const float* vy;              // [T][H][W] MC variance of y
  int32_t K;                    // candidates
  double scale[kMaxBandwidths]; // h / h_k (the plan's h over the candidate)
  double h[kMaxBandwidths];     // candidate bandwidths
  float* hsel;                  // [n_out] nullable
  float* sure;                  // [n_out] nullable
};

hipError_t launch_log_variance(const float* E, const float* var, float* vy, int64_t n, int spp, float eps,
                               hipStream_t s);
// lanes: 16 (work lists, small frames) or 1 (dense).
hipError_t launch_bandwidth(const BandwidthArgs& b, int F, bool f16, int lanes, const DeviceShape& dev,
                            hipStream_t s);

}  // namespace esim
