// Shared by the two fitness routers: the normalisation of Eq. 5.
#pragma once

#include <hip/hip_runtime.h>

namespace maestro {

// (x - lo) / (hi - lo) clipped to [0, 1]; 0 for a degenerate window
__device__ __forceinline__ float norm01(float x, float lo, float hi) {
  if (!(hi > lo)) return 0.0f;
  float t = __fdiv_rn(__fsub_rn(x, lo), __fsub_rn(hi, lo));
  if (t < 0.0f) t = 0.0f;
  if (t > 1.0f) t = 1.0f;
  return t;
}

}  // namespace maestro
