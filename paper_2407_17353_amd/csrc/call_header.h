// Workspace header of a matmul call, device side: the exponents every
// workgroup derives from the scales, and the header's life within one call
// without a kernel that clears it first.
//
// Workgroup 0 claims, clears and publishes the header once its first loads
// are under way, so that the others, which use it at their end, find it ready;
// a workgroup that comes there before it has, does so in its place
// (header_tag.h: nothing depends on the order of dispatch). Whoever ends the
// call's use of the header takes the tag out again:
//   single pass: the first workgroup, once every workgroup has arrived (or,
//     after an abort, the last one to have written its tiles);
//   direct cast with a statistic: the last workgroup to arrive;
//   GEMM + cast kernel: the cast kernel.
//
// Output scale and statistic are written only after every workgroup has
// arrived, so they may share memory with an input scale or with amax_in.
#pragma once
#include "codec.h"
#include "header_tag.h"
#include "kernels.h"

namespace scalify {

// Header words (see kernels.h).
// Words 0 .. 31 share a cache line that only sees atomics while workgroups
// arrive (11 ns each, one after the other); what is polled lies in the other
// line, as a load of a line under atomics costs all of them some 50 ns.
constexpr int kHdrArrive = 5, kHdrState = 6, kHdrWritten = 7, kHdrTag = 32, kHdrGo = 34;
enum SpState : uint32_t { SP_RUNNING = 0, SP_COMPLETE = 1, SP_ABORTED = 2 };

// What a workgroup derives from the scales: the pre-cast value's exponent,
// the shifts of a residual add (Algorithm 3), and (direct cast) the output's
// exponent and shift.
struct CallExponents {
  int e_w;     // true value of w is w * 2^e_w
  int sh_acc;  // accumulator into w's scale
  int sh_res;  // residual into w's scale
  int e_out;   // direct cast
  int shift;   // direct cast: data' = w * 2^-shift
};

// The scales' bits, loaded at the start of the kernel (scalar loads without a
// branch: a NULL scale reads the output scale's word and is then 1) and
// turned into exponents where they are first needed.
struct RawScales {
  uint32_t s0, s1, s_res, amax_in;
};

__device__ __forceinline__ RawScales load_scales(const GemmParams& p) {
  const uint32_t one = 0x3F800000u;
  auto word = [&](const float* q, uint32_t dflt) {
    const uint32_t v = *(const uint32_t*)(q ? q : p.out_scale);
    return q ? v : dflt;
  };
  return RawScales{word(p.s0, one), word(p.s1, one), word(p.s_res, one), word(p.amax_in, 0u)};
}

// Exponent of a power of two given by its fp32 bits (normal or subnormal).
__device__ __forceinline__ int pow2_exponent_bits(uint32_t u) {
  const int e = (int)((u >> 23) & 0xFFu);
  if (e != 0) return e - 127;
  const uint32_t m = u & 0x7FFFFFu;
  return m ? (31 - __clz((int)m)) - 149 : -127;
}

__device__ __forceinline__ CallExponents call_exponents(const GemmParams& p, const RawScales& r) {
  CallExponents x;
  const int e_ab = pow2_exponent_bits(r.s0) + pow2_exponent_bits(r.s1);
  x.e_w = e_ab;
  x.sh_acc = x.sh_res = 0;
  if (p.residual) {
    // sqrt(2^(2 e_p) + 2^(2 e_q)) rounded down to a power of two is the
    // larger of the two scales
    const int e_q = pow2_exponent_bits(r.s_res);
    x.e_w = max(e_ab + p.e_c, e_q);
    x.sh_acc = e_ab - x.e_w;
    x.sh_res = e_q - x.e_w;
  }
  x.e_out = x.shift = 0;
  if (p.epi == EPI_DIRECT) {
    // |statistic| of an earlier call (delayed rescale), or none (e_r = 0)
    x.e_out = clamp_e8m0(x.e_w + p.e_cc + rescale_exponent(r.amax_in & 0x7FFFFFFFu, p.target));
    x.shift = x.e_out - x.e_w;
  }
  return x;
}

__device__ __forceinline__ void hdr_store(uint32_t* q, uint32_t v) {
  __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t hdr_load(uint32_t* q) {
  return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t* hdr_tag(const GemmParams& p) {
  return (uint64_t*)(p.hdr + kHdrTag);
}

// The header's words as a call starts with them.
__device__ __forceinline__ void header_clear(const GemmParams& p, int e_w) {
  hdr_store(p.hdr, 0u);
  hdr_store(p.hdr + 1, (uint32_t)e_w);
  hdr_store(p.hdr + kHdrArrive, 0u);
  hdr_store(p.hdr + kHdrState, (uint32_t)SP_RUNNING);
  hdr_store(p.hdr + kHdrGo, (uint32_t)SP_RUNNING);
  hdr_store(p.hdr + kHdrWritten, 0u);
}
// Workgroup 0, one thread, with its first loads under way (the claim waits for
// them): whether it has claimed the header; its words are then on their way
// and header_publish follows, the same thread, after a wait that covers them
// (vector memory completes in issue order).
__device__ __forceinline__ bool header_begin(const GemmParams& p, const RawScales& r) {
  if (!tag_claim(hdr_tag(p), p.tag)) return false;
  header_clear(p, call_exponents(p, r).e_w);
  return true;
}
__device__ __forceinline__ void header_publish(const GemmParams& p) { tag_store(hdr_tag(p), p.tag); }
// Both, where the kernel has nothing to do in between.
__device__ __forceinline__ void header_open(const GemmParams& p, const RawScales& r) {
  if (!header_begin(p, r)) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  header_publish(p);
}
__device__ __forceinline__ void header_retire(const GemmParams& p) { tag_store(hdr_tag(p), 0); }
// One thread of a workgroup, before its first use of the header.
__device__ __forceinline__ void header_await(const GemmParams& p, int e_w) {
  tag_await(hdr_tag(p), p.tag, [&] {
    header_clear(p, e_w);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  });
}

// Fold the workgroup's statistic and count its arrival: returns how many have
// arrived, this one included (the max is performed before the count).
__device__ __forceinline__ uint32_t header_arrive(const GemmParams& p, float wmax) {
  __hip_atomic_fetch_max(p.hdr, __float_as_uint(wmax), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  return __hip_atomic_fetch_add(p.hdr + kHdrArrive, 1u, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT) + 1u;
}

// End of a workgroup of the direct cast, one thread: with a statistic to
// report (or an output scale that shares memory with an input), the last
// workgroup to arrive writes both; else workgroup 0 writes the scale.
__device__ __forceinline__ void direct_finish(const GemmParams& p, float wmax, int G,
                                              const CallExponents& x) {
  if (p.counted) {
    header_await(p, x.e_w);
    if (header_arrive(p, wmax) != (uint32_t)G) return;
    if (p.amax_out)
      *p.amax_out = __uint_as_float(hdr_load(p.hdr)) * pow2_float(-p.e_cc);
    header_retire(p);
    *p.out_scale = pow2_float(x.e_out);
  } else if (blockIdx.x == 0) {
    *p.out_scale = pow2_float(x.e_out);
  }
}

// End of a workgroup of the GEMM that leaves the cast to a kernel of its own.
__device__ __forceinline__ void pair_finish(const GemmParams& p, float wmax, int e_w) {
  header_await(p, e_w);
  atomicMax(p.hdr, __float_as_uint(wmax));
}

// Grid barrier of the single pass on the statistic, one thread of a workgroup.
// grid_arrive folds the workgroup's max and counts its arrival; the last
// arrival sets the go word COMPLETE. grid_wait waits for that, bounded
// (p.spin_ticks of the 100 MHz real-time counter): a workgroup that runs out
// sets ABORTED unless the word has changed; whichever of the two is set
// first decides for every workgroup (and is recorded in the state word).
// word[0]: the decision, word[1]: the statistic (of everyone, after COMPLETE).
__device__ __forceinline__ uint32_t grid_decide(const GemmParams& p, uint32_t decision) {
  uint32_t e = SP_RUNNING;
  __hip_atomic_compare_exchange_strong(p.hdr + kHdrGo, &e, decision, __ATOMIC_RELAXED,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (e != SP_RUNNING) return e;
  hdr_store(p.hdr + kHdrState, decision);
  return decision;
}

__device__ __forceinline__ uint32_t grid_arrive(const GemmParams& p, float wmax, int G,
                                                int e_w) {
  header_await(p, e_w);
  if (header_arrive(p, wmax) != (uint32_t)G) return SP_RUNNING;
  return grid_decide(p, SP_COMPLETE);
}

__device__ __forceinline__ void grid_wait(const GemmParams& p, uint32_t st, uint32_t* word) {
  // (a poll takes at least the sleep, 256 cycles: the poll count bounds the
  // wait even if the counter did not advance)
  if (st == SP_RUNNING) st = hdr_load(p.hdr + kHdrGo);
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  const int64_t max_polls = p.spin_ticks + 64;
  for (int64_t it = 0; st == SP_RUNNING && it < max_polls &&
                       (int64_t)(__builtin_amdgcn_s_memrealtime() - t0) < p.spin_ticks;
       ++it) {
    __builtin_amdgcn_s_sleep(4);
    st = hdr_load(p.hdr + kHdrGo);
  }
  if (st == SP_RUNNING) st = grid_decide(p, SP_ABORTED);
  word[0] = st;
  word[1] = hdr_load(p.hdr);
  if (st == SP_COMPLETE && blockIdx.x == 0) header_retire(p);  // (everyone has arrived)
}

// After an abort, once this workgroup's tiles are in the intermediate: counts
// it and tells whether it was the last (which then casts every tile, from
// everyone's stores and with the statistic of all).
__device__ __forceinline__ bool last_writer(const GemmParams& p, int G, uint32_t* word,
                                            uint32_t& amax_raw) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t w = __hip_atomic_fetch_add(p.hdr + kHdrWritten, 1u, __ATOMIC_ACQ_REL,
                                              __HIP_MEMORY_SCOPE_AGENT) + 1u;
    word[0] = w == (uint32_t)G ? 1u : 0u;
    word[1] = hdr_load(p.hdr);
    if (w == (uint32_t)G) header_retire(p);
  }
  __syncthreads();
  amax_raw = word[1];
  if (!word[0]) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return true;
}

// Shift of the cast from the amax statistic (bits of max |w|): the rescale
// exponent of Section 3.3 rounded down, e_out = clamp(e_w + e_cc + e_r).
__device__ __forceinline__ int sp_shift(uint32_t amax_raw, int e_w, int e_cc, int target,
                                        int* e_out_p) {
  int e_r = 0;
  if (amax_raw != 0u && amax_raw < 0x7F800000u) e_r = floor_log2_bits(amax_raw) - e_cc - target;
  const int e_out = clamp_e8m0(e_w + e_cc + e_r);
  *e_out_p = e_out;
  return e_out - e_w;
}

}  // namespace scalify
