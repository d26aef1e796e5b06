// The LayerNorm's row kernels that read each row from HBM once.
//
// What bounds them: HBM, once the arithmetic is kept below it. The row's
// values are decoded once and kept (as x, then x - mean, in place); a lane
// holds 32 of them, so the sums, divisions and the square root that every
// lane does per row cost little per element, and three waves per SIMD still
// fit (two with FP32 inputs, and in the backward with FP16 or FP32 gradients),
// which keep the next rows' loads in flight (the kernels before these
// re-decoded 64 raw elements per lane in each of four passes and were bound by
// that: backward of 16384 x 4096, F16 x and E5M2 dy, 112 us, 98 us now).
//
// A row of D <= 2048 columns belongs to one wave, of up to 4096 to two and of
// up to 8192 to four waves of a workgroup (WPR); wave part k takes the lane
// chunks 2 k and 2 k + 1 (part order of layernorm_dev.h), and the parts' sums
// meet in LDS. The raw codes of the next row of the workgroup's stride are
// loaded while a row is computed. FULL: D = 2048 WPR, every chunk whole.
#pragma once
#include "layernorm_dev.h"

namespace scalify {

// Sum of the parts of a row (values of WPR waves), in part order, to every
// lane of them: v is the wave's own part sum. slot: [rows of the workgroup][WPR].
template <int WPR, int NV>
__device__ __forceinline__ void row_sum(float (&v)[NV], float (*slot)[WPR][NV], int row, int part,
                                        int lane) {
  if constexpr (WPR > 1) {
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) slot[row][part][i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float s = slot[row][0][i];
#pragma unroll
      for (int k = 1; k < WPR; ++k) s += slot[row][k][i];
      v[i] = s;
    }
  }
}

// This lane's two chunks of a row: first columns, valid elements (may be <= 0).
template <int WPR, bool FULL>
struct RowChunks {
  int n[2], valid[2];
  __device__ __forceinline__ RowChunks(int D, int part, int lane) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      n[j] = 16 * (lane + 64 * (2 * part + j));
      valid[j] = FULL ? 16 : D - n[j];
    }
  }
};

template <int F>
__device__ __forceinline__ void load_row(const void* base, int64_t row_off, bool row_ok,
                                         const int (&n)[2], const int (&valid)[2],
                                         uint32_t (&w)[2][ln_chunk_words<F>()]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) ln_load_raw<F>(base, row_off + n[j], row_ok ? valid[j] : 0, w[j]);
}

// The parameters of a lane's columns (they are the same for every row).
template <bool FULL>
__device__ __forceinline__ void load_params(const float* p, float dflt, const int (&n)[2],
                                            const int (&valid)[2], float (&v)[2][16]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) ln_param16(p, n[j], FULL ? 16 : max(valid[j], 0), dflt, v[j]);
}

// x -> x - mean in place, with the row's mean and standard deviation.
template <int WPR, bool FULL>
__device__ __forceinline__ void center_row(float (&x)[2][16], const int (&valid)[2], int D,
                                           float (*slot1)[WPR][1], float (*slot2)[WPR][1], int row,
                                           int part, int lane, float& mu, float& sigma) {
#pragma clang fp contract(off)
  float cs[2] = {0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) cs[j] += x[j][i];  // columns >= D are 0
  float s[1] = {wave_sum(cs[0] + cs[1])};
  row_sum<WPR, 1>(s, slot1, row, part, lane);
  mu = s[0] / (float)D;
  float ct[2] = {0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float d = x[j][i] - mu;
      x[j][i] = FULL || i < valid[j] ? d : 0.0f;
      ct[j] = fmaf(x[j][i], d, ct[j]);  // (one rounding per term)
    }
  float t[1] = {wave_sum(ct[0] + ct[1])};
  row_sum<WPR, 1>(t, slot2, row, part, lane);
  sigma = sqrtf(t[0] / (float)D);
}

template <int XF, int OUTF, int WPR, bool FULL>
__global__ __launch_bounds__(LN_THREADS) void ln_fwd_rows_kernel(LnParams p) {
  // (no FMA contraction: the fused multiply-adds are written out, the same
  // in the single-read and multi-pass kernels, so both round alike)
#pragma clang fp contract(off)
  constexpr int RPW = 4 / WPR;  // rows of a workgroup
  __shared__ float s1[RPW][WPR][1], s2[RPW][WPR][1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = wave / WPR, part = wave % WPR;
  const bool sat = p.sat != 0;
  const RowChunks<WPR, FULL> ch(p.D, part, lane);
  if (blockIdx.x == 0 && threadIdx.x == 0) *p.out_scale = 1.0f;  // Appendix C.2: scale 1
  const int64_t stride = (int64_t)gridDim.x * RPW;
  uint32_t w[2][ln_chunk_words<XF>()];
  int64_t r0 = (int64_t)blockIdx.x * RPW;
  load_row<XF>(p.x, (r0 + slot) * p.ldx, r0 + slot < p.R, ch.n, ch.valid, w);
  float gam[2][16], bet[2][16];
  load_params<FULL>(p.gamma, 1.0f, ch.n, ch.valid, gam);
  load_params<FULL>(p.beta, 0.0f, ch.n, ch.valid, bet);
#pragma unroll 1
  for (; r0 < p.R; r0 += stride) {
    const int64_t r = r0 + slot;
    float x[2][16];
#pragma unroll
    for (int j = 0; j < 2; ++j) ln_decode16<XF>(w[j], x[j]);
    load_row<XF>(p.x, (r + stride) * p.ldx, r + stride < p.R, ch.n, ch.valid, w);
    float mu, sigma;
    center_row<WPR, FULL>(x, ch.valid, p.D, s1, s2, slot, part, lane, mu, sigma);
    const float inv = 1.0f / (sigma + p.eps);
    if (r < p.R) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (!FULL && ch.valid[j] <= 0) continue;
        float y[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) y[i] = fmaf(x[j][i] * inv, gam[j][i], bet[j][i]);
        if (p.pre_out) ln_store_f32(p.pre_out + r * (int64_t)p.D + ch.n[j], ch.valid[j], y);
        ln_store16<OUTF>(p.out, r * p.ldo + ch.n[j], ch.valid[j], y, 0, 1.0f, true, sat);
      }
    }
  }
}

// Waves per SIMD that the backward's registers are held to: three, which the
// compiler misses by a few registers when left alone (F16 x, E5M2 dy, 32768 x
// 2512: 276 us with two), where they fit without spills.
template <int XF, int DYF, bool FULL>
constexpr int ln_bwd_waves() {
  return XF != kF32 && (DYF == kE4M3 || DYF == kE5M2 || (DYF == kF16 && FULL)) ? 3 : 2;
}

// The backward's statistics: the four numbers of every row (rowstats) and the
// amax of |dx|, with ln_dx's arithmetic. The last multiplication of dx, by
// 1 / (std + eps) > 0, keeps the order of magnitudes, so it is done once per
// row and lane, on the largest factor. The call's header: stat_header.h.
template <int XF, int DYF, int WPR, bool FULL>
__global__ __launch_bounds__(LN_THREADS, (ln_bwd_waves<XF, DYF, FULL>())) void ln_bwd_rows_kernel(LnParams p) {
  // (no FMA contraction: see ln_fwd_rows_kernel)
#pragma clang fp contract(off)
  constexpr int RPW = 4 / WPR;
  __shared__ float s1[RPW][WPR][1], s2[RPW][WPR][1], s3[RPW][WPR][2];
  __shared__ float wmax[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = wave / WPR, part = wave % WPR;
  const RowChunks<WPR, FULL> ch(p.D, part, lane);
  float4* rowstats = (float4*)p.partial;
  const int64_t stride = (int64_t)gridDim.x * RPW;
  uint32_t wx[2][ln_chunk_words<XF>()], wd[2][ln_chunk_words<DYF>()];
  int64_t r0 = (int64_t)blockIdx.x * RPW;
  load_row<XF>(p.x, (r0 + slot) * p.ldx, r0 + slot < p.R, ch.n, ch.valid, wx);
  load_row<DYF>(p.dy, (r0 + slot) * p.lddy, r0 + slot < p.R, ch.n, ch.valid, wd);
  float gam[2][16];
  load_params<FULL>(p.gamma, 1.0f, ch.n, ch.valid, gam);
  if (blockIdx.x == 0 && threadIdx.x == 0) stat_open(p.hdr, p.tag, p.s_dy, p.s_x);
  float lmax = 0.0f;
#pragma unroll 1
  for (; r0 < p.R; r0 += stride) {
    const int64_t r = r0 + slot;
    float x[2][16], g[2][16];
#pragma unroll
    for (int j = 0; j < 2; ++j) ln_decode16<XF>(wx[j], x[j]);
    load_row<XF>(p.x, (r + stride) * p.ldx, r + stride < p.R, ch.n, ch.valid, wx);
    float mu, sigma;
    center_row<WPR, FULL>(x, ch.valid, p.D, s1, s2, slot, part, lane, mu, sigma);
    const float inv = 1.0f / (sigma + p.eps);
    float cg[2] = {0.0f, 0.0f}, cx[2] = {0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ln_decode16<DYF>(wd[j], g[j]);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        g[j][i] = g[j][i] * gam[j][i];
        if (!FULL) g[j][i] = i < ch.valid[j] ? g[j][i] : 0.0f;
        cg[j] += g[j][i];
        cx[j] = fmaf(g[j][i], x[j][i] * inv, cx[j]);
      }
    }
    load_row<DYF>(p.dy, (r + stride) * p.lddy, r + stride < p.R, ch.n, ch.valid, wd);
    float s[2] = {wave_sum(cg[0] + cg[1]), wave_sum(cx[0] + cx[1])};
    row_sum<WPR, 2>(s, s3, slot, part, lane);
    float4 st;
    st.x = mu;
    st.y = inv;
    st.z = s[0] / (float)p.D;
    st.w = sigma > 0.0f ? (s[1] / (float)p.D) / sigma : 0.0f;
    if (r < p.R) {
      if (lane == 0 && part == 0) rowstats[r] = st;
      float tmax = 0.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float t[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          t[i] = g[j][i] - st.z - x[j][i] * st.w;  // dx is t * st.y
          if (FULL || i < ch.valid[j]) tmax = fmaxf(tmax, fabsf(t[i]));  // fmaxf skips NaN
        }
        if (p.pre_out && (FULL || ch.valid[j] > 0)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) t[i] *= st.y;
          ln_store_f32(p.pre_out + r * (int64_t)p.D + ch.n[j], ch.valid[j], t);
        }
      }
      lmax = fmaxf(lmax, tmax * st.y);
    }
  }
  // amax of |dx|: wave butterfly, then the four waves, then the header
  for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
  if (lane == 0) wmax[wave] = lmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    stat_await(p.hdr, p.tag, p.s_dy, p.s_x);
    stat_fold(p.hdr, fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
  }
}

}  // namespace scalify
