// Order-preserving keys of routing logits, shared by the selection kernels of
// dynamic.hip and dyntop.hip.
#pragma once

#include "moce_internal.h"

namespace moce {

// Order-preserving key of a float (larger float, larger key); -0 is taken as
// +0 first, so that equal logits have equal keys.
__device__ __forceinline__ uint32_t fkey(float v) {
  const uint32_t u = __float_as_uint(v + 0.f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);   // negative: every bit inverted
}
__device__ __forceinline__ float fkey_value(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

}  // namespace moce
