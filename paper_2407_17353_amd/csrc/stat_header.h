// Workspace header of the calls whose statistic one kernel gathers and the
// next one reads (rescale, LayerNorm backward), without a kernel that clears
// it first: workgroup 0 opens the header at its start, or whoever needs it
// before that (header_tag.h), the others fold their statistic in, and the
// kernel that reads the statistic takes the tag out again.
// Words: [0] amax bits, [1] scale exponent snapshot, [32..33] tag.
#pragma once
#include "codec.h"
#include "header_tag.h"

namespace scalify {

constexpr int kStatTag = 32;  // (not in the line of the atomics: a load of that line costs them 50 ns each)

__device__ __forceinline__ uint64_t* stat_tag(uint32_t* hdr) { return (uint64_t*)(hdr + kStatTag); }

// Clear the statistic and take the snapshot of the scale exponent
// e(s0) - e(s1) (an output scale may share their memory).
__device__ __forceinline__ void stat_clear(uint32_t* hdr, const float* s0, const float* s1) {
  __hip_atomic_store(hdr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(hdr + 1, (uint32_t)(pow2_exponent(s0) - pow2_exponent(s1)), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// Workgroup 0, one thread, at its start.
__device__ __forceinline__ void stat_open(uint32_t* hdr, uint64_t tag, const float* s0, const float* s1) {
  if (!tag_claim(stat_tag(hdr), tag)) return;
  stat_clear(hdr, s0, s1);
  tag_store(stat_tag(hdr), tag);
}
// One thread of a workgroup, before its first fold.
__device__ __forceinline__ void stat_await(uint32_t* hdr, uint64_t tag, const float* s0, const float* s1) {
  tag_await(stat_tag(hdr), tag, [&] { stat_clear(hdr, s0, s1); });
}
// Fold a maximum in; returns the largest of the others' so far.
__device__ __forceinline__ float stat_fold(uint32_t* hdr, float wmax) {
  return __uint_as_float(__hip_atomic_fetch_max(hdr, __float_as_uint(wmax), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT));
}
// One thread of the kernel that reads the statistic.
__device__ __forceinline__ void stat_retire(uint32_t* hdr) { *stat_tag(hdr) = 0; }

}  // namespace scalify
