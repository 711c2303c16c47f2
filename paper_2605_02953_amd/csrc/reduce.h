// Eight bf16 values of a 16-byte vector in fp32: taken, added, and rounded back once.
#pragma once
#include "common.h"

namespace ditron {

__device__ __forceinline__ void set_bf16x8(float (&acc)[8], const u32x4_t v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[2 * j] = __builtin_bit_cast(float, v[j] << 16);
    acc[2 * j + 1] = __builtin_bit_cast(float, v[j] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ void add_bf16x8(float (&acc)[8], const u32x4_t v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[2 * j] += __builtin_bit_cast(float, v[j] << 16);
    acc[2 * j + 1] += __builtin_bit_cast(float, v[j] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ u32x4_t pack_bf16x8(const float (&acc)[8]) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  u32x4_t r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bf16x2_t v = {(__bf16)acc[2 * j], (__bf16)acc[2 * j + 1]};
    r[j] = __builtin_bit_cast(uint32_t, v);
  }
  return r;
}

}  // namespace ditron
