// Internal interface between the C ABI (scalify_abi.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scalify {

// Workspace header, in 32-bit words at the start of every workspace
// (call_header.h: its life within a matmul call; stat_header.h: of the
// rescale and the LayerNorm backward, words 0, 1, 32 and 33):
//   [0] amax as fp32 bits (atomic max target)
//   [1] e_w, the scale exponent of the pre-cast value w (the exponent sum of
//       the input scales, or the scaled-add exponent with a residual)
//   [5] workgroups that have folded their maximum in
//   [6] single pass: barrier state, 0 running, 1 complete, 2 aborted
//   [7] single pass: workgroups that wrote their held tile after an abort
//   [32] and [33] the call's tag while the header is in use
//   [34] single pass: the barrier's decision, polled
constexpr size_t kHeaderBytes = 256;

// Activation of the fused epilogue (values of scalify_activation).
enum Act : int { ACT_NONE = 0, ACT_RELU = 1, ACT_GELU_TANH = 2, ACT_SILU = 3 };

// What the GEMM writes: a pre-cast intermediate for the cast kernel that
// follows (16-bit rounding-preserving encoding for FP8 outputs, the fp32
// accumulator for FP16 outputs), or, when the output scale is known before
// the GEMM runs (delayed rescale), the output codes themselves.
enum Epi : int { EPI_INTER16 = 0, EPI_INTER32 = 1, EPI_DIRECT = 2 };

struct GemmParams {
  const uint8_t* a;
  const uint8_t* b;
  int64_t lda, ldb;
  uint32_t a_bytes, b_bytes;  // stored-matrix sizes (buffer range limits)
  int M, N, K;
  int tiles_m, tiles_n;
  int e_c;        // matmul scale rule exponent
  int e_cc;       // exponent offset of the statistic: e_c, or 0 with a residual
  const float* s0;       // scales of a, b and the residual (NULL = 1)
  const float* s1;
  const float* s_res;
  const float* amax_in;  // delayed rescale: the statistic of an earlier call
  uint64_t tag;          // of this call (call_header.h)
  int uses_header;       // the call needs the header's words
  int counted;           // direct cast: the last workgroup writes scale and statistic
  int residual;          // scaled add of a residual (whose data may be empty)
  int sat;
  uint32_t* hdr;  // workspace header
  void* inter;    // pre-cast intermediate [M][ldw] (EPI_INTER16: u16, EPI_INTER32: f32)
  int64_t ldw;
  float* acc_out;  // optional raw accumulator [M][N]
  void* out;       // EPI_DIRECT: output codes [M][ldc] of format out_fmt
  int64_t ldc;
  int out_fmt;
  // Fused epilogue: residual codes [M][ldr] (ldr = 0:
  // one row for every row) of format res_fmt or NULL, activation, and the
  // optional export of the pre-cast value w [M][N].
  const void* res;
  int64_t ldr;
  int res_fmt;
  int act;
  float* pre_out;
  // Channel scales: powers of two per output row
  // (ch_a [M]) and per output column (ch_b [N]) multiplied into the
  // accumulator with the power-of-two product of the epilogue; NULL = 1.
  const float* ch_a;
  const float* ch_b;
  // MX block scales (MX kernels only), packed by launch_mx_pack: per 128-k
  // step and 64-row group (mx_groups_* = ceil(rows / 64) groups), 64 words,
  // word 16 g + r holding the bytes of rows r, r + 16, r + 32, r + 48 of the
  // group at k-block g of the step; byte sizes for the buffer range checks.
  const uint8_t* mx_a;
  const uint8_t* mx_b;
  int mx_groups_a, mx_groups_b;
  uint32_t mx_a_bytes, mx_b_bytes;
  // The persistent 4-wave kernel: workgroups (gemm4_grid), and the single
  // pass of the dynamic rescale (EPI_INTER16 / EPI_INTER32 kernels that hold
  // their last tile, meet at a grid barrier and cast): its rescale target,
  // the output scale and statistic it writes, and the barrier's wait budget
  // in ticks of the 100 MHz real-time counter.
  int grid;
  int epi;  // Epi of the launch
  int single_pass;
  int target;
  float* out_scale;
  float* amax_out;
  int64_t spin_ticks;
};

// Workgroups of the persistent 4-wave kernel for `tiles` output tiles: one
// per CU of the current device (its LDS holds one workgroup), at most one
// per tile.
int gemm4_grid(int tiles);

// Packed MX block scales (see GemmParams) from row-major bytes src[r * ld + b].
hipError_t launch_mx_pack(const uint8_t* src, int rows, int K, int ld, uint8_t* dst,
                          hipStream_t s);

hipError_t launch_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb, hipStream_t s);

// The 256 x 256 kernel with the fused epilogue (one workgroup per tile).
hipError_t launch_fused_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb,
                             hipStream_t s);

// Header of a rescale without a statistic: hdr[0] = 0, hdr[1] = exponent(s0)
// (NULL = scale 1).
hipError_t launch_prologue(uint32_t* hdr, const float* s0, hipStream_t s);

// A matmul with no output elements: output scale and statistic alone.
struct EmptyMatmul {
  const float* s0;
  const float* s1;
  const float* s_res;    // residual scale (NULL = 1)
  int residual, e_c;
  const float* amax_in;  // delayed rescale, else NULL
  int target;
  float* out_scale;
  float* amax_out;       // or NULL
};
hipError_t launch_empty_matmul(const EmptyMatmul& q, hipStream_t s);

// Cast of the GEMM intermediate [M][ldw] to out [M][ldc]; computes the
// rescale exponent from hdr and writes *out_scale (and *amax_out).
struct EpilogueParams {
  const void* inter;
  int64_t ldw;
  void* out;
  int64_t ldc;
  int M, N;
  int e_c, target, sat, mode;
  uint32_t* hdr;  // (its tag is taken out: the call is done with the header)
  float* out_scale;
  float* amax_out;
};
hipError_t launch_epilogue_cast(const EpilogueParams& p, int inter32, int out_dtype,
                                hipStream_t s);

// Elementwise rescale / cast / set_scaling of a contiguous array of n elements.
enum ScaleRule : int { RULE_AMAX = 0, RULE_KEEP = 1, RULE_FIXED = 2, RULE_COPY = 3 };
struct ElemParams {
  const void* in;
  void* out;
  int64_t n;
  int rule;          // RULE_AMAX: from hdr amax; RULE_KEEP: e_out = e_in; RULE_FIXED: e_out = e_fixed;
                     // RULE_COPY: shift 0 and the raw input scale value is copied
  int target, sat, e_fixed;
  uint32_t* hdr;            // RULE_AMAX (whose tag is taken out), RULE_KEEP (e_in snapshot) or NULL
  const float* in_scale;    // read directly when hdr is NULL
  float* out_scale;
};
// The header's statistic and exponent snapshot of in_scale (stat_header.h).
hipError_t launch_amax(const void* in, int in_dtype, int64_t n, const float* in_scale, uint32_t* hdr,
                       uint64_t tag, hipStream_t s);
hipError_t launch_elementwise(const ElemParams& p, int in_dtype, int out_dtype, hipStream_t s);

}  // namespace scalify
