// Order of the DA-FPS pick's values as two 32-bit words, compared high word
// first (signed), then low word (unsigned): the order of the doubles.  A
// negative value has the bits of both halves of its magnitude inverted, so
// the larger magnitude comes lower in either; no value is -0.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace apack {

__host__ __device__ __forceinline__ uint64_t double_bits(double v) {
  uint64_t b;
  __builtin_memcpy(&b, &v, 8);
  return b;
}
__host__ __device__ __forceinline__ int pick_key_high(double v) {
  const int h = (int)(double_bits(v) >> 32);
  return h ^ ((h >> 31) & 0x7FFFFFFF);
}
__host__ __device__ __forceinline__ uint32_t pick_key_low(double v) {
  const uint64_t b = double_bits(v);
  return (uint32_t)b ^ (uint32_t)((int)(b >> 32) >> 31);
}
// The product of a value's two factors, a zero one (also one that underflows)
// as +0.
__host__ __device__ __forceinline__ double pick_value(double a, double b) { return fma(a, b, 0.0) + 0.0; }

}  // namespace apack
