// The workspace header's protocol (csrc/header_tag.h) on the CPU: workgroups
// as calls or threads, in any order, on a header with any contents.
// Prints "ok" and returns 0, or says what failed.
#include <cstdio>
#include <cstring>
#include <random>
#include <thread>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_store(q, v, order, scope) __atomic_store_n(q, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_load(q, order, scope) __atomic_load_n(q, __ATOMIC_SEQ_CST)
#define __hip_atomic_compare_exchange_strong(q, e, v, o1, o2, scope) \
  __atomic_compare_exchange_n(q, e, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)
// A wait that sleeps this often in a row has no one left to wait for.
static thread_local long sleeps = 0;
static long max_sleeps = 0;
struct Stuck {};
static void nap() {
  if (++sleeps > max_sleeps) throw Stuck{};
  std::this_thread::yield();
}
#define __builtin_amdgcn_s_sleep(n) nap()
#include "../paper_2407_17353_amd/csrc/header_tag.h"

struct Header {
  uint64_t tag;
  uint32_t amax, arrived;
};

struct Call {
  Header* h;
  uint64_t tag;
  uint32_t groups;
  uint32_t result = 0, clears = 0, finished = 0;

  void clear() {
    __atomic_store_n(&h->amax, 0u, __ATOMIC_SEQ_CST);
    __atomic_store_n(&h->arrived, 0u, __ATOMIC_SEQ_CST);
    __atomic_fetch_add(&clears, 1u, __ATOMIC_SEQ_CST);
  }
  // A workgroup as the kernels run it: workgroup 0 tries to clear the header
  // at its start; everyone folds its value in and counts itself at its end,
  // and the last one reads the result and takes the tag out.
  void start(uint32_t g, bool& owned) {
    owned = g == 0 && scalify::tag_claim(&h->tag, tag);
    if (owned) clear();
  }
  void end(uint32_t g, bool owned) {
    if (owned) scalify::tag_store(&h->tag, tag);
    sleeps = 0;
    scalify::tag_await(&h->tag, tag, [&] { clear(); });
    uint32_t v = value(g), seen = __atomic_load_n(&h->amax, __ATOMIC_SEQ_CST);
    while (seen < v && !__atomic_compare_exchange_n(&h->amax, &seen, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {
    }
    if (__atomic_add_fetch(&h->arrived, 1u, __ATOMIC_SEQ_CST) != groups) return;
    result = __atomic_load_n(&h->amax, __ATOMIC_SEQ_CST);
    __atomic_fetch_add(&finished, 1u, __ATOMIC_SEQ_CST);
    scalify::tag_store(&h->tag, 0);
  }
  uint32_t value(uint32_t g) const { return 1u + (uint32_t)((tag >> 7) * 2654435761u + g * 40503u) % 100000u; }
  bool check(const char* what) const {
    uint32_t want = 0;
    for (uint32_t g = 0; g < groups; ++g) want = value(g) > want ? value(g) : want;
    if (clears == 1 && finished == 1 && result == want && h->tag == 0) return true;
    printf("%s: clears %u finished %u result %u want %u tag %llx\n", what, clears, finished, result, want,
           (unsigned long long)h->tag);
    return false;
  }
};

// What a header may hold when a call starts: zeros, a fill, the leftovers of
// another call (its tag or its claim), all ones.
static void fill(Header& h, int kind) {
  memset(&h, kind == 1 ? 0xAB : (kind == 4 ? 0xFF : 0), sizeof h);
  if (kind == 2) h = Header{0x123456789ABCDEF0ull, 7u, 3u};
  if (kind == 3) h = Header{0x123456789ABCDEF1ull, 0xFFFFFFFFu, 2u};
}

int main() {
  std::mt19937_64 rng(1);
  Header h;
  try {
    // One workgroup after the other, workgroup 0 first, in the middle or last
    // (its start only after others have ended): nobody may wait for it.
    max_sleeps = 0;
    for (int kind = 0; kind < 5; ++kind)
      for (uint32_t groups : {1u, 2u, 7u})
        for (uint32_t zero_at = 0; zero_at < groups; ++zero_at) {
          fill(h, kind);
          Call c{&h, rng() & ~1ull, groups};
          for (int replay = 0; replay < 3; ++replay) {
            c.clears = c.finished = c.result = 0;
            for (uint32_t i = 0; i < groups; ++i) {
              const uint32_t g = i == zero_at ? 0u : (i < zero_at ? i + 1 : i);
              bool owned;
              c.start(g, owned);
              c.end(g, owned);
            }
            if (!c.check("sequential")) return 1;
          }
        }
    // Workgroup 0 has claimed the header but not published it: its own end
    // does, whoever came in between finds it claimed.
    fill(h, 1);
    Call c{&h, rng() & ~1ull, 1};
    bool owned, again;
    c.start(0, owned);
    if (!owned || scalify::tag_claim(&h.tag, c.tag)) return puts("claimed twice"), 1;
    c.start(0, again);
    if (again) return puts("claimed again"), 1;
    c.end(0, owned);
    if (!c.check("claimed early")) return 1;
  } catch (Stuck&) {
    return puts("a workgroup waits for one that has not run"), 1;
  }
  // Threads, in the order the machine runs them.
  max_sleeps = 1l << 40;
  for (int rep = 0; rep < 300; ++rep) {
    fill(h, rep % 5);
    Call c{&h, rng() & ~1ull, 8};
    std::vector<std::thread> t;
    for (uint32_t i = 0; i < 8; ++i)
      t.emplace_back([&c, g = (i + rep) % 8] {
        bool owned;
        c.start(g, owned);
        c.end(g, owned);
      });
    for (auto& x : t) x.join();
    if (!c.check("threads")) return 1;
  }
  puts("ok");
  return 0;
}
