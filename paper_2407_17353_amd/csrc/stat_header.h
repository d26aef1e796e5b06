// Workspace header of the calls whose statistic one kernel gathers and the
// next one reads (rescale, LayerNorm backward), without a kernel that clears
// it first. The host draws a 64-bit tag for every call:
// workgroup 0 clears the words and publishes the call's tag, the others fold
// their statistic in once they have seen it, and the kernel that reads the
// statistic takes the tag out again (a replay of a captured call carries the
// same tag). Words: [0] amax bits, [1] scale exponent snapshot, [32..33] tag.
#pragma once
#include "codec.h"

namespace scalify {

constexpr int kStatTag = 32;  // (not in the line of the atomics: a load of that line costs them 50 ns each)

// Workgroup 0, one thread: clear the statistic and take the snapshot of the
// scale exponent e(s0) - e(s1) (an output scale may share their memory).
__device__ __forceinline__ void stat_clear(uint32_t* hdr, const float* s0, const float* s1) {
  __hip_atomic_store(hdr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(hdr + 1, (uint32_t)(pow2_exponent(s0) - pow2_exponent(s1)), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
// The same thread, later: the stores above are done, publish the tag.
__device__ __forceinline__ void stat_publish(uint32_t* hdr, uint64_t tag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __hip_atomic_store((uint64_t*)(hdr + kStatTag), tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One thread of a workgroup: wait for the tag. (Workgroup 0 is never
// dispatched after the others and publishes at its start, so the wait ends;
// the poll count, seconds of polling, only makes that unconditional.)
__device__ __forceinline__ void stat_await(uint32_t* hdr, uint64_t tag) {
  for (int it = 0; it < (1 << 22); ++it) {
    if (__hip_atomic_load((uint64_t*)(hdr + kStatTag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag)
      return;
    __builtin_amdgcn_s_sleep(2);
  }
}
// Fold a maximum in; returns the largest of the others' so far.
__device__ __forceinline__ float stat_fold(uint32_t* hdr, float wmax) {
  return __uint_as_float(__hip_atomic_fetch_max(hdr, __float_as_uint(wmax), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT));
}
// One thread of the kernel that reads the statistic.
__device__ __forceinline__ void stat_retire(uint32_t* hdr) { *(uint64_t*)(hdr + kStatTag) = 0; }

}  // namespace scalify
