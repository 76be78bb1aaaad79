// One-kernel backward of the weighted product at equal degrees 1..8
// (gtp_wbwd.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gtp {

struct WbwdArgs {
  const void *x1, *x2;         // [n, K] of in_type
  int in_type;
  const float* dy;             // [n, K]
  const float *w1, *w2, *wo;   // [R, L + 1] or null (ones); R = C with per_channel, else 1
  float *dx1, *dx2;            // [n, K] or null
  float *dw1, *dw2, *dwo;      // [R, L + 1] or null
  float* partial;              // wbwd_partial_floats, or null when no weight gradient is asked for
  int64_t n, C, waves;         // products, channels, wbwd_waves
  int per_channel;
  int need;                    // 1: dwo, 2: dx1 or dw1, 4: dx2 or dw2, 16: dw1, 32: dw2
};

// Workgroups (of one wave) of the kernel, and the floats of its partial sums.
int64_t wbwd_waves(int64_t n, int64_t C, int per_channel);
int64_t wbwd_partial_floats(int L, int64_t waves, int per_channel);
hipError_t launch_wbwd_small(int L, const WbwdArgs& a, hipStream_t s, bool* supported);

}  // namespace gtp
