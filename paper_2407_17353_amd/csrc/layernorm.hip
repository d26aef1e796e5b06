// Scaled LayerNorm (Appendix C.2) and its input gradient with the dynamic
// rescale (the LayerNorm backward rescale of the experiments, Section 4).
//
// Forward: a mean-variance normalization is scale invariant up to its eps,
// so the data component X_d is normalized and the output gets scale 1:
//   xhat = (x - mean) / (std + eps),  y = xhat * gamma + beta,  cast(y).
// Backward: the gradient with respect to X_d, as the ScaledArray
// (dx, s_dy / s_x), then rebalanced by the amax rule and cast:
//   dx = (g - mean(g) - (c / std) mean(g * xhat)) / (std + eps),  g = dy * gamma,
//   c = x - mean; dgamma = sum_rows dy * xhat, dbeta = sum_rows dy.
//
// The row kernels (layernorm_rows.h) read each row once; the multi-pass
// kernels here give the same bits and run when SCALIFY_LN_SINGLE_READ=0 asks
// for them. The backward's statistic kernel keeps, per row, the four numbers
// dx needs; its apply kernel is then a streaming pass over 32-row x
// 2048-column tiles that casts dx with the rescale the global amax gives and
// accumulates the tile's partial parameter gradients, which a last kernel
// sums over the row tiles in a fixed order.
#include "kernels.h"
#include "layernorm_dev.h"

#include <stdlib.h>

namespace scalify {

// A row's sum in the order of layernorm_dev.h: chunk(q) is the sum of chunk q.
template <typename F>
__device__ __forceinline__ float ln_row_sum(int D, int lane, F&& chunk) {
#pragma clang fp contract(off)
  const int nch = (D + 15) / 16;
  float total = 0.0f;
#pragma unroll 1
  for (int k = 0; k < nch; k += 128) {
    const float c0 = k + lane < nch ? chunk(k + lane) : 0.0f;
    const float c1 = k + lane + 64 < nch ? chunk(k + lane + 64) : 0.0f;
    const float part = wave_sum(c0 + c1);
    total = k ? total + part : part;
  }
  return total;
}

// Mean and std of row r: two passes over the row, the second one served by
// the caches (fp32, the order of layernorm_dev.h).
template <int XF>
__device__ __forceinline__ void ln_row_stats(const LnParams& p, int64_t r, int lane, float& mu,
                                             float& sigma) {
  // (no FMA contraction: the fused multiply-adds are written out, the same
  // in the single-read and multi-pass kernels, so both round alike)
#pragma clang fp contract(off)
  mu = ln_row_sum(p.D, lane, [&](int q) {
    float v[16], cs = 0.0f;
    ln_chunk_f<XF>(p.x, r * p.ldx + 16 * q, p.D - 16 * q, v);
#pragma unroll
    for (int i = 0; i < 16; ++i) cs += v[i];  // columns >= D read as 0
    return cs;
  }) / (float)p.D;
  const float m = mu;
  const float t = ln_row_sum(p.D, lane, [&](int q) {
    float v[16], ct = 0.0f;
    const int valid = p.D - 16 * q;
    ln_chunk_f<XF>(p.x, r * p.ldx + 16 * q, valid, v);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float d = v[i] - m;
      ct = fmaf(i < valid ? d : 0.0f, d, ct);  // (one rounding per term)
    }
    return ct;
  });
  sigma = sqrtf(t / (float)p.D);
}

template <int XF, int OUTF>
__global__ __launch_bounds__(LN_THREADS) void ln_fwd_kernel(LnParams p) {
  // (no FMA contraction: the fused multiply-adds are written out, the same
  // in the single-read and multi-pass kernels, so both round alike)
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const bool sat = p.sat != 0;
  const int nch = (p.D + 15) / 16;
  if (blockIdx.x == 0 && threadIdx.x == 0) *p.out_scale = 1.0f;  // Appendix C.2: scale 1
#pragma unroll 1
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < p.R; r += (int64_t)gridDim.x * 4) {
    float mu, sigma;
    ln_row_stats<XF>(p, r, lane, mu, sigma);
    const float inv = 1.0f / (sigma + p.eps);
#pragma unroll 1
    for (int q = lane; q < nch; q += 64) {
      const int n = 16 * q;
      const int valid = p.D - n;
      float v[16], g[16], b[16], y[16];
      ln_chunk_f<XF>(p.x, r * p.ldx + n, valid, v);
      ln_param16(p.gamma, n, valid, 1.0f, g);
      ln_param16(p.beta, n, valid, 0.0f, b);
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = fmaf((v[i] - mu) * inv, g[i], b[i]);
      if (p.pre_out) ln_store_f32(p.pre_out + r * (int64_t)p.D + n, valid, y);
      ln_store16<OUTF>(p.out, r * p.ldo + n, valid, y, 0, 1.0f, true, sat);
    }
  }
}

template <int XF>
__global__ __launch_bounds__(LN_THREADS) void ln_bwd_stats_kernel(LnParams p) {
  // (no FMA contraction: the fused multiply-adds are written out, the same
  // in the single-read and multi-pass kernels, so both round alike)
#pragma clang fp contract(off)
  __shared__ float wmax[4];
  if (blockIdx.x == 0 && threadIdx.x == 0) stat_open(p.hdr, p.tag, p.s_dy, p.s_x);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nch = (p.D + 15) / 16;
  float lmax = 0.0f;
  float4* rowstats = (float4*)p.partial;
#pragma unroll 1
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < p.R; r += (int64_t)gridDim.x * 4) {
    float mu, sigma;
    ln_row_stats<XF>(p, r, lane, mu, sigma);
    const float inv = 1.0f / (sigma + p.eps);
    // (two sums over the same passes: the second one re-reads the row)
    auto product = [&](int q, bool with_x) {
      const int n = 16 * q;
      const int valid = p.D - n;
      float v[16], d[16], gam[16], c = 0.0f;
      ln_chunk_f<XF>(p.x, r * p.ldx + n, valid, v);
      ln_load16(p.dy_fmt, p.dy, r * p.lddy + n, valid, d);
      ln_param16(p.gamma, n, valid, 1.0f, gam);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float g = i < valid ? d[i] * gam[i] : 0.0f;
        const float e = i < valid ? v[i] - mu : 0.0f;
        c = with_x ? fmaf(g, e * inv, c) : c + g;
      }
      return c;
    };
    const float sg = ln_row_sum(p.D, lane, [&](int q) { return product(q, false); });
    const float sgx = ln_row_sum(p.D, lane, [&](int q) { return product(q, true); });
    float4 st;
    st.x = mu;
    st.y = inv;
    st.z = sg / (float)p.D;
    st.w = sigma > 0.0f ? (sgx / (float)p.D) / sigma : 0.0f;
    if (lane == 0) rowstats[r] = st;
#pragma unroll 1
    for (int q = lane; q < nch; q += 64) {
      const int n = 16 * q;
      const int valid = p.D - n;
      float v[16], d[16], gam[16], dx[16];
      ln_chunk_f<XF>(p.x, r * p.ldx + n, valid, v);
      ln_load16(p.dy_fmt, p.dy, r * p.lddy + n, valid, d);
      ln_param16(p.gamma, n, valid, 1.0f, gam);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        dx[i] = ln_dx(v[i], d[i], gam[i], st);
        if (i < valid) lmax = fmaxf(lmax, fabsf(dx[i]));  // fmaxf skips NaN
      }
      if (p.pre_out) ln_store_f32(p.pre_out + r * (int64_t)p.D + n, valid, dx);
    }
  }
  // amax of |dx|: wave butterfly, the four waves, one atomic max per workgroup
  for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
  if (lane == 0) wmax[wave] = lmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    stat_await(p.hdr, p.tag, p.s_dy, p.s_x);
    stat_fold(p.hdr, fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
  }
}

// dgamma[j], dbeta[j] = fixed-order sums of the row tiles' partials: a
// workgroup covers 64 columns; its LN_PARAM_WAVES waves sum interleaved
// shares of the tiles (wave w: tiles w, w + LN_PARAM_WAVES, ...), then wave
// 0 adds the wave sums pairwise in a fixed tree. (Few columns, many tiles:
// the waves of a workgroup keep more of the tiles' loads in flight.)
constexpr int LN_PARAM_WAVES = 16;

__global__ __launch_bounds__(64 * LN_PARAM_WAVES) void ln_params_kernel(const float* part, int tiles,
                                                                        int D, float* dgamma,
                                                                        float* dbeta) {
  __shared__ float red[2][LN_PARAM_WAVES][64];
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + c;
  const int64_t dp = layernorm_param_stride(D);
  float g = 0.0f, b = 0.0f;
  if (j < D) {
#pragma unroll 8
    for (int k = w; k < tiles; k += LN_PARAM_WAVES) {
      g += part[(int64_t)k * 2 * dp + j];
      b += part[(int64_t)k * 2 * dp + dp + j];
    }
  }
  red[0][w][c] = g;
  red[1][w][c] = b;
  __syncthreads();
  if (w == 0 && j < D) {
    float sg[LN_PARAM_WAVES], sb[LN_PARAM_WAVES];
#pragma unroll
    for (int i = 0; i < LN_PARAM_WAVES; ++i) {
      sg[i] = red[0][i][c];
      sb[i] = red[1][i][c];
    }
#pragma unroll
    for (int h = 1; h < LN_PARAM_WAVES; h *= 2)
#pragma unroll
      for (int i = 0; i < LN_PARAM_WAVES; i += 2 * h) {
        sg[i] += sg[i + h];
        sb[i] += sb[i + h];
      }
    if (dgamma) dgamma[j] = sg[0];
    if (dbeta) dbeta[j] = sb[0];
  }
}

// Without rows: the output scale and a statistic of 0. (The workspace, which
// may then have no bytes at all, is not touched.)
__global__ void ln_bwd_empty_kernel(const float* s_dy, const float* s_x, float* out_scale, float* amax_out) {
  if (threadIdx.x == 0) {
    *out_scale = pow2_float(clamp_e8m0(pow2_exponent(s_dy) - pow2_exponent(s_x)));
    if (amax_out) *amax_out = 0.0f;
  }
}

static int row_grid(int64_t R) {
  const int64_t b = (R + 3) / 4;
  return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

int64_t layernorm_row_tiles(int64_t R) {
  const int64_t t = (R + LN_TILE_ROWS - 1) / LN_TILE_ROWS;
  return t < 1 ? 1 : t;
}

int64_t layernorm_ws_floats(int64_t R, int64_t D) {
  return 4 * R + layernorm_row_tiles(R) * 2 * layernorm_param_stride(D);
}

// Workgroups of the row kernels: at most per_cu per CU, each walking rows with
// the grid's stride.
int ln_rows_grid(int64_t R, int wpr, int per_cu) {
  const int rpw = 4 / wpr;
  const int64_t need = (R + rpw - 1) / rpw;
  const int64_t g = (int64_t)per_cu * gemm4_grid(1 << 30);  // (CUs of the current device)
  return (int)(need < 1 ? 1 : (need < g ? need : g));
}

// The single-read kernels unless SCALIFY_LN_SINGLE_READ=0 (read at each
// call), which takes the multi-pass ones for every width.
static bool single_read_enabled() {
  const char* v = getenv("SCALIFY_LN_SINGLE_READ");
  return !(v && v[0] == '0' && v[1] == 0);
}

template <int XF>
static void launch_fwd_xf(const LnParams& p, int out_dtype, hipStream_t s) {
  if (single_read_enabled()) return launch_ln_fwd_rows<XF>(p, out_dtype, s);
  const dim3 g(row_grid(p.R)), b(LN_THREADS);
  if (out_dtype == kE4M3) hipLaunchKernelGGL((ln_fwd_kernel<XF, kE4M3>), g, b, 0, s, p);
  else if (out_dtype == kE5M2) hipLaunchKernelGGL((ln_fwd_kernel<XF, kE5M2>), g, b, 0, s, p);
  else hipLaunchKernelGGL((ln_fwd_kernel<XF, kF16>), g, b, 0, s, p);
}

hipError_t launch_layernorm_fwd(const LnParams& p, int out_dtype, hipStream_t s) {
  if (p.x_fmt == kF16) launch_fwd_xf<kF16>(p, out_dtype, s);
  else if (p.x_fmt == kF32) launch_fwd_xf<kF32>(p, out_dtype, s);
  else if (p.x_fmt == kE4M3) launch_fwd_xf<kE4M3>(p, out_dtype, s);
  else launch_fwd_xf<kE5M2>(p, out_dtype, s);
  return hipGetLastError();
}

template <int XF>
static void launch_bwd_xf(const LnParams& p, int out_dtype, hipStream_t s) {
  if (single_read_enabled())
    launch_ln_bwd_rows<XF>(p, s);
  else
    hipLaunchKernelGGL((ln_bwd_stats_kernel<XF>), dim3(row_grid(p.R)), dim3(LN_THREADS), 0, s, p);
  launch_ln_apply<XF>(p, out_dtype, s);
}

hipError_t launch_layernorm_bwd(const LnParams& p, int out_dtype, hipStream_t s) {
  if (p.R == 0)
    hipLaunchKernelGGL(ln_bwd_empty_kernel, dim3(1), dim3(64), 0, s, p.s_dy, p.s_x, p.out_scale, p.amax_out);
  else if (p.x_fmt == kF16) launch_bwd_xf<kF16>(p, out_dtype, s);
  else if (p.x_fmt == kF32) launch_bwd_xf<kF32>(p, out_dtype, s);
  else if (p.x_fmt == kE4M3) launch_bwd_xf<kE4M3>(p, out_dtype, s);
  else launch_bwd_xf<kE5M2>(p, out_dtype, s);
  if ((p.dgamma || p.dbeta) && p.D > 0)
    hipLaunchKernelGGL(ln_params_kernel, dim3((p.D + 63) / 64), dim3(64 * LN_PARAM_WAVES), 0, s,
                       p.partial + 4 * p.R,
                       p.R ? (int)layernorm_row_tiles(p.R) : 0, p.D, p.dgamma, p.dbeta);
  return hipGetLastError();
}

}  // namespace scalify
