// bfloat16 as the warm-start network stores it: the upper half of an FP32
// value, rounded to nearest even (NaN stays NaN).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mfbd {

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// (a select and no branch: a kernel converts whole rows of values)
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  return (uint16_t)(f == f ? r : (u >> 16) | 0x40u);
}

}  // namespace mfbd
