// The exact power-of-two scaling of keys shared by the key preparation and the similarity sweep, and
// the similarities that the sweep's packed values stand for.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace twinkv {

// Power of two g with ||g k|| in (0.5, 1] given r = 1/||k|| (1 for zero or bad keys).
__device__ inline float row_scale(float r) {
  if (!(r > 0.0f) || !(r < 3.0e38f)) return 1.0f;
  int e;
  (void)frexpf(r, &e);
  return ldexpf(1.0f, e - 1);
}

// Multiply 8 bf16 values by a power of two.  Exact unless a value leaves the normal range.
__device__ inline uint4 scale_bf16x8(uint4 raw, float g) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float lo = __uint_as_float(w[k] << 16) * g;
    const float hi = __uint_as_float(w[k] & 0xFFFF0000u) * g;
    o[k] = (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xFFFF0000u);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

constexpr uint32_t kValidMin = 0x3F800000u;  // packed values >= 1.0f are real candidates

// The similarity that a packed value x stands for, for a token of inverse norm ri.
__device__ inline float similarity(uint32_t x, float ri) {
  return (__uint_as_float(x) - 3.0f) * ri / row_scale(ri);
}

}  // namespace twinkv
