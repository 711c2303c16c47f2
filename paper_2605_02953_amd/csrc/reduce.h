// The sum of `world` bf16 blocks in fp32, slot after slot, rounded once: what GEMM-ReduceScatter ends with, as a launch of its
// own (reduce_slots_kernel) or as the last work-groups of another one (MoE down-projection + ReduceScatter).
#pragma once
#include "common.h"

namespace ditron {

struct ReduceParams {
  const void* slot[DITRON_MAX_WORLD];
  const int32_t* gate[DITRON_MAX_WORLD];  // first flag of slot s (chunk c at gate[s] + c*gate_stride[s]) or null
  int gate_stride[DITRON_MAX_WORLD];
  __bf16* out;
  int32_t* status;
  size_t vec_per_chunk;  // 16-byte vectors per row chunk
  int chunks, world;
  int32_t epoch;
  unsigned spin_limit;
  int wgs_per_chunk;
};

constexpr int kReduceUnroll = 1;     // 16-byte vectors per lane per slot in flight

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

// Work-group `wg` of p.chunks * p.wgs_per_chunk, THREADS threads.  WORLD > 0 fixes the number of slots at compile time (fully
// unrolled slot loop).
template <int WORLD, int THREADS>
__device__ __forceinline__ void reduce_slots_work_group(const ReduceParams& p, int wg) {
  const int chunk = wg / p.wgs_per_chunk;
  const int part = wg % p.wgs_per_chunk;
  const int world = WORLD > 0 ? WORLD : p.world;
  // one lane per slot: the flags are looked at side by side, not one round trip after another
  if ((int)threadIdx.x < world && p.gate[threadIdx.x])
    flag_wait_lane(p.gate[threadIdx.x], chunk * p.gate_stride[threadIdx.x], 1, p.epoch, p.spin_limit, p.status);
  __syncthreads();
  const size_t base = (size_t)chunk * p.vec_per_chunk;
  const size_t step = (size_t)p.wgs_per_chunk * THREADS;
  u32x4_t* out = (u32x4_t*)p.out + base;
  size_t i = (size_t)part * THREADS + threadIdx.x;
  for (; i + (kReduceUnroll - 1) * step < p.vec_per_chunk; i += kReduceUnroll * step) {
    float acc[kReduceUnroll][8];
    {
      u32x4_t v[kReduceUnroll];
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u)
        v[u] = __builtin_nontemporal_load((const u32x4_t*)p.slot[0] + base + i + u * step);
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u) set_bf16x8(acc[u], v[u]);
    }
#pragma unroll
    for (int s = 1; s < world; ++s) {
      u32x4_t v[kReduceUnroll];
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u)
        v[u] = __builtin_nontemporal_load((const u32x4_t*)p.slot[s] + base + i + u * step);
#pragma unroll
      for (int u = 0; u < kReduceUnroll; ++u) add_bf16x8(acc[u], v[u]);
    }
#pragma unroll
    for (int u = 0; u < kReduceUnroll; ++u) __builtin_nontemporal_store(pack_bf16x8(acc[u]), out + i + u * step);
  }
  for (; i < p.vec_per_chunk; i += step) {
    float acc[8];
    set_bf16x8(acc, ((const u32x4_t*)p.slot[0])[base + i]);
    for (int s = 1; s < world; ++s) add_bf16x8(acc, ((const u32x4_t*)p.slot[s])[base + i]);
    out[i] = pack_bf16x8(acc);
  }
}

}  // namespace ditron
