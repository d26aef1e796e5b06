// The LayerNorm backward's second kernel: dx cast with the rescale that the
// statistic gives, and the partial parameter gradients.
#pragma once
#include "layernorm_dev.h"

namespace scalify {

// Tile (row block blockIdx.y of LN_TILE_ROWS rows, column block blockIdx.x of
// LN_TILE_COLS columns): dx recomputed from the row numbers, cast with the
// rescale, and the tile's partial parameter gradients.
template <int XF, int DYF, int OUTF>
__global__ __launch_bounds__(LN_TILE_THREADS) void ln_bwd_apply_kernel(LnParams p) {
  const int e_in = (int)p.hdr[1];
  int e_r = 0;
  if (p.mode == 1) e_r = rescale_exponent(p.hdr[0], p.target);
  const int e_out = clamp_e8m0(e_in + e_r);
  const int shift = e_out - e_in;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    *p.out_scale = pow2_float(e_out);
    if (p.amax_out) *p.amax_out = __uint_as_float(p.hdr[0]);
    stat_retire(p.hdr);
  }
  const bool sat = p.sat != 0;
  const bool fast = shift >= kFastShiftMinSub && shift <= kFastShiftMax;
  const float scale = fast ? pow2_float(shift) : 1.0f;
  const int n = (int)blockIdx.x * LN_TILE_COLS + 16 * (int)threadIdx.x;
  const int valid = p.D - n;
  // The rows that the statistic's kernel read last are still in the last-level
  // cache: they are taken first.
  const int tile = (int)(gridDim.y - 1 - blockIdx.y);
  const float4* rowstats = (const float4*)p.partial;
  const int64_t dp = layernorm_param_stride(p.D);
  float* part = p.partial + 4 * p.R + (int64_t)tile * 2 * dp;
  if (valid <= 0) return;
  float gam[16], pg[16], pb[16];
  ln_param16(p.gamma, n, valid, 1.0f, gam);
#pragma unroll
  for (int i = 0; i < 16; ++i) pg[i] = pb[i] = 0.0f;
  const int64_t r0 = (int64_t)tile * LN_TILE_ROWS;
  const int64_t r1 = r0 + LN_TILE_ROWS < p.R ? r0 + LN_TILE_ROWS : p.R;
  // The rows' raw codes go through a ring of PF slots: slot k holds row
  // rb + k while it is computed and then receives row rb + k + PF, so PF
  // rows' loads are in flight while one is computed (the per-row sums keep
  // their row order).
  constexpr int PF = 4;
  uint32_t rx[PF][ln_chunk_words<XF>()], rd[PF][ln_chunk_words<DYF>()];
#pragma unroll
  for (int k = 0; k < PF; ++k)
    if (r0 + k < r1) {
      ln_load_raw<XF>(p.x, (r0 + k) * p.ldx + n, valid, rx[k]);
      ln_load_raw<DYF>(p.dy, (r0 + k) * p.lddy + n, valid, rd[k]);
    }
#pragma unroll 1
  for (int64_t rb = r0; rb < r1; rb += PF) {
    ln_static_for<0, PF>([&](auto K) {
      constexpr int k = decltype(K)::value;
      const int64_t r = rb + k;
      if (r < r1) {
        const float4 st = rowstats[r];
        float dx[16];
        float xv[16], dv[16];
        ln_decode16<XF>(rx[k], xv);
        ln_decode16<DYF>(rd[k], dv);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float x = xv[i], d = dv[i];
          dx[i] = ln_dx(x, d, gam[i], st);
          pg[i] += d * ((x - st.x) * st.y);
          pb[i] += d;
        }
        ln_store16<OUTF>(p.out, r * p.ldo + n, valid, dx, shift, scale, fast, sat);
        if (r + PF < r1) {
          ln_load_raw<XF>(p.x, (r + PF) * p.ldx + n, valid, rx[k]);
          ln_load_raw<DYF>(p.dy, (r + PF) * p.lddy + n, valid, rd[k]);
        }
      }
    });
  }
  if (p.dgamma || p.dbeta) {
    ln_store_f32(part + n, valid, pg);
    ln_store_f32(part + dp + n, valid, pb);
  }
}

}  // namespace scalify
