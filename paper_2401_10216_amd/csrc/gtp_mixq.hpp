// Sample-domain channel mixing at equal degrees 1..8 (gtp_mixq.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gtp {

struct MixqArgs {
  const void *x1, *x2;  // [B, C1, K], [B, C2, K] of in_type; the matrix cores contract over C1
  int in_type;
  const float* W;       // W[co C1 C2 + c1 s1 + c2 s2]
  int64_t s1, s2;
  void* work;           // the weights' operand images and exponents (mixq_work_bytes)
  float* y;             // [B, Co, K]
  int64_t B, C1, C2, Co;
};

// Size of MixqArgs::work.
int64_t mixq_work_bytes(int64_t Co, int64_t C1, int64_t C2);
hipError_t launch_mixq(int L, const MixqArgs& a, hipStream_t s, bool* supported);

}  // namespace gtp
