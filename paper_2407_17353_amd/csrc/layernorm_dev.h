// Device helpers of the scaled LayerNorm kernels (layernorm_*.hip): element
// access, wave sums and the order in which a row is summed.
//
// Order of a row's sums, the same in every kernel (so the single-read and the
// multi-pass ones give the same bits): lane l takes the 16-column chunks l,
// l + 64, ...; two neighbouring chunks of a lane make a part (128 chunks, 2048
// columns, per part): the chunk sums are added, the part's 64 lane values are
// summed by a butterfly, and the parts are added in order.
#pragma once
#include "codec.h"
#include "ew_util.h"
#include "layernorm.h"
#include "stat_header.h"

#include <type_traits>

namespace scalify {

// f(std::integral_constant<int, I>), ..., up to N - 1 (compile-time indices).
template <int I, int N, typename F>
__device__ __forceinline__ void ln_static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    ln_static_for<I + 1, N>(f);
  }
}

constexpr int LN_THREADS = 256;   // 4 waves: 4 rows at a time
constexpr int LN_TILE_ROWS = 32;  // apply kernel: rows per workgroup
constexpr int LN_TILE_THREADS = 128;
constexpr int LN_TILE_COLS = 16 * LN_TILE_THREADS;

template <int F>
__device__ __forceinline__ void ln_chunk_f(const void* base, int64_t off, int valid,
                                           float (&v)[16]) {
  uint32_t c[16];
  if (valid >= 16) {
    load16<F>(base, off, c);
  } else {
    // ragged end of the row: element loads at clamped (valid) addresses
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = load1<F>(base, off + (i < valid ? i : 0));
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = i < valid ? decode_hw<F>(c[i]) : 0.0f;
}

// 16 values of a row from column n (columns >= D read as 0), format fmt.
__device__ __forceinline__ void ln_load16(int fmt, const void* base, int64_t off, int valid,
                                          float (&v)[16]) {
  if (fmt == kF16) ln_chunk_f<kF16>(base, off, valid, v);
  else if (fmt == kE4M3) ln_chunk_f<kE4M3>(base, off, valid, v);
  else if (fmt == kE5M2) ln_chunk_f<kE5M2>(base, off, valid, v);
  else ln_chunk_f<kF32>(base, off, valid, v);
}

__device__ __forceinline__ void ln_param16(const float* p, int n, int valid, float dflt,
                                           float (&v)[16]) {
  if (p == nullptr || valid <= 0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = dflt;
  } else if (valid >= 16) {
    ln_chunk_f<kF32>(p, n, 16, v);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = i < valid ? p[n + i] : dflt;
  }
}

// Sum over the wave, the same bits in every lane: a butterfly over lane
// distances 1, 2, 4, 8 (DPP), 16 and 32 (lane swaps), no LDS round trips.
__device__ __forceinline__ float wave_sum(float a) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                      0xF, 0xF, true));
  };
  a += dpp(a, std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
  a += dpp(a, std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
  a += dpp(a, std::integral_constant<int, 0x141>{});  // row_half_mirror: the other quad of 8
  a += dpp(a, std::integral_constant<int, 0x140>{});  // row_mirror: the other half of 16
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  a = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Cast and store 16 values of one row at column n.
template <int OUTF>
__device__ __forceinline__ void ln_store16(void* out, int64_t off, int valid, const float (&y)[16],
                                           int shift, float scale, bool fast, bool sat) {
  uint32_t u[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) u[i] = __float_as_uint(y[i]);
  uint32_t w[8];
  encode16<OUTF>(u, shift, scale, fast, sat, w);
  if (valid >= 16) {
    store_words16<OUTF>(out, off, w);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i < valid) store1<OUTF>(out, off + i, word_code<OUTF>(w, i));
  }
}

__device__ __forceinline__ void ln_store_f32(float* q, int valid, const float (&y)[16]) {
  if (valid >= 16 && ((uintptr_t)q & 15u) == 0) {
#pragma unroll
    for (int h = 0; h < 4; ++h) *(u4*)(q + 4 * h) = u4{__float_as_uint(y[4 * h]), __float_as_uint(y[4 * h + 1]),
                                                         __float_as_uint(y[4 * h + 2]), __float_as_uint(y[4 * h + 3])};
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i < valid) q[i] = y[i];
  }
}

template <int XF>
__device__ __forceinline__ float ln_raw_decode(const uint32_t* w, int i) {
  if constexpr (XF == kF32) return __uint_as_float(w[i]);
  else if constexpr (XF == kF16) return decode_hw<kF16>((w[i >> 1] >> (16 * (i & 1))) & 0xFFFFu);
  else return decode_hw<XF>((w[i >> 2] >> (8 * (i & 3))) & 0xFFu);
}

// The 16 elements of a chunk's raw codes as fp32 (exact), FP8 codes two per
// conversion (the packed form takes the low or the high 16 bits of a word).
template <int XF>
__device__ __forceinline__ void ln_decode16(const uint32_t* w, float (&x)[16]) {
  if constexpr (XF == kE4M3 || XF == kE5M2) {
    auto pk = [](uint32_t v, auto hi_tag) {
      if constexpr (XF == kE4M3)
        return __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(v, 1.0f, decltype(hi_tag)::value);
      else
        return __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(v, 1.0f, decltype(hi_tag)::value);
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const auto lo = pk(w[k], std::false_type{});
      const auto hi = pk(w[k], std::true_type{});
      x[4 * k] = lo[0];
      x[4 * k + 1] = lo[1];
      x[4 * k + 2] = hi[0];
      x[4 * k + 3] = hi[1];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = ln_raw_decode<XF>(w, i);
  }
}

// Dwords of a 16-element chunk of format F, and the chunk's raw codes at
// element e of base (valid elements, the rest zero: codes that decode to 0; a
// lane past the row's end has none and skips the chunk). The loads are 16 bytes
// wide also where the row ends inside one: rows are 16-byte aligned, so a load
// that holds an element of the row stays in the row's padding (ld).
// (Element loads there, whose sixteen tests every wave went through for the
// lanes past the end as well, took the forward of 16384 x 512 F16 25 us, the
// backward of 16384 x 2512 F16 147; now 16 and 99.)
template <int F>
constexpr int ln_chunk_words() { return F == kF32 ? 16 : (F == kF16 ? 8 : 4); }

template <int F>
__device__ __forceinline__ void ln_load_raw(const void* base, int64_t e, int valid,
                                            uint32_t (&w)[ln_chunk_words<F>()]) {
  constexpr int W = ln_chunk_words<F>();
  constexpr int EPW = 16 / W;  // elements per dword
#pragma unroll
  for (int k = 0; k < W; ++k) w[k] = 0u;
  auto piece = [&](int h) {
    const u4 v = F == kF32 ? *((const u4*)((const uint32_t*)base + e) + h)
                           : (F == kF16 ? *((const u4*)((const uint16_t*)base + e) + h)
                                        : *((const u4*)((const uint8_t*)base + e) + h));
#pragma unroll
    for (int k = 0; k < 4; ++k) w[4 * h + k] = v[k];
  };
  if (valid >= 16) {
#pragma unroll
    for (int h = 0; h < W / 4; ++h) piece(h);
  } else if (valid > 0) {
#pragma unroll
    for (int h = 0; h < W / 4; ++h)
      if (valid > 4 * EPW * h) piece(h);
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const int n = valid - EPW * k;  // elements of dword k
      w[k] = n <= 0 ? 0u : (n >= EPW ? w[k] : w[k] & ((1u << (32 / EPW * n & 31)) - 1u));
    }
  }
}

// Per-row numbers of the gradient (rowstats[r] = {mean, 1/(std+eps), mean(g),
// mean(g * xhat)/std or 0}), so that dx = (dy gamma - mean(g) - (x - mean) t) * inv.
// Both backward kernels evaluate it with this code and no contraction, so the
// apply kernel casts bit for bit the values whose amax the statistic measured.
__device__ __forceinline__ float ln_dx(float x, float dy, float gam, const float4& st) {
#pragma clang fp contract(off)
  const float g = dy * gam;
  return (g - st.z - (x - st.x) * st.w) * st.y;
}

}  // namespace scalify
