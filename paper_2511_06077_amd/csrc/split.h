// Exchange between the workgroups that divide a target group's hidden layer
// (fast.hip, bwd_update.hip, paper.hip).
#pragma once

#include "common.h"

namespace stca {

// Each of `splits` workgroups of group `group` (of `groups`) holds its part v
// of a 32-target tile, 16 values a thread, NT threads.  Leaves it in spart
// ([splits][groups][16 NT] floats) and counts its arrival in *cnt (zero
// before); true in the last workgroup to arrive, whose v is then the sum of
// the parts in split order, whoever is last.  The parts are in register order
// (the reader's thread holds the same elements), so every access of a wave is
// one contiguous 512-byte piece, and go through agent-scope relaxed atomics:
// stores that write through to memory, waited for before the arrival is
// counted, and loads that bypass the XCD's L2.  (Agent-scope fences write
// back and invalidate a whole L2 instead, once a wave, and cost more than the
// work that was split.)  `arrived`: a shared variable of the workgroup.
template <int NT>
__device__ __forceinline__ bool split_sum(f32x16& v, float* spart, int32_t* cnt, int splits, int groups, int group,
                                          int split, int* arrived) {
  auto part_at = [&](int k, int i) {
    return reinterpret_cast<uint64_t*>(spart) + (((int64_t)k * groups + group) * 8 + i) * NT + threadIdx.x;
  };
#pragma unroll
  for (int i = 0; i < 8; ++i)
    __hip_atomic_store(part_at(split, i),
                       (uint64_t)__float_as_uint(v[2 * i]) | ((uint64_t)__float_as_uint(v[2 * i + 1]) << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the part is in memory before its arrival is counted
  __syncthreads();
  if (threadIdx.x == 0) *arrived = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (*arrived != splits - 1) return false;
  v = f32x16{};
  for (int k = 0; k < splits; ++k)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint64_t x = __hip_atomic_load(part_at(k, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[2 * i] += __uint_as_float(static_cast<uint32_t>(x));
      v[2 * i + 1] += __uint_as_float(static_cast<uint32_t>(x >> 32));
    }
  return true;
}

}  // namespace stca
