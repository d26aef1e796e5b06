// Who clears a workspace header, and when the others may use it.
//
// The workspace arrives with any contents, and no order in which workgroups
// are dispatched is promised (each XCD starts its own share of a grid, and
// another stream's kernel may hold the CUs of one of them). The header's tag
// word therefore decides: the host draws an even 64-bit tag for every call;
// whichever workgroup claims the word first (compare-and-swap to tag | 1)
// clears the header and then stores the tag itself. A workgroup uses the
// header only once it has seen the tag, and claims it if nobody has. It waits
// for nobody but a claimant, which is running and waits for no one until it
// has published, so the wait ends whatever the dispatch order.
//
// Whoever ends the call's use of the header stores 0, so that a replay of the
// same launch (which carries the same tag) starts like the first one.
#pragma once
#include <stdint.h>

namespace scalify {

constexpr uint64_t kTagClaimed = 1;

__device__ __forceinline__ void tag_store(uint64_t* word, uint64_t v) {
  __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One thread: whether it is the one that clears the header and then, once
// those stores are done, publishes the tag with tag_store(word, tag).
__device__ __forceinline__ bool tag_claim(uint64_t* word, uint64_t tag) {
  uint64_t seen = 0;  // (what an earlier call leaves: one round trip)
  while (!__hip_atomic_compare_exchange_strong(word, &seen, tag | kTagClaimed, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    if (seen == tag || seen == (tag | kTagClaimed)) return false;
  }
  return true;
}

// One thread of a workgroup, before its first use of the header. clear() is
// the header's clearing, its stores complete when it returns.
template <typename Clear>
__device__ __forceinline__ void tag_await(uint64_t* word, uint64_t tag, Clear&& clear) {
  for (;;) {
    const uint64_t seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (seen == tag) return;
    if (seen != (tag | kTagClaimed) && tag_claim(word, tag)) {
      clear();
      tag_store(word, tag);
      return;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

}  // namespace scalify
