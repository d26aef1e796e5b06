// Epilogue of the GEMM kernels whose threads take groups of 4 consecutive
// outputs of a row (mid_gemm_kernel.h, wave_gemm_kernel.h), in batches of NB
// groups of one thread: columns n .. n + 3 of the rows m, m + dm, m + 2 dm, ...
//
// Every choice that is the same for the whole call (residual format,
// activation, output format, saturation) is made once per batch, outside the
// loop over its groups, so that the loads, conversions and stores of a batch
// are straight-line code and overlap; a choice per group cost 7 us of a
// 128 x 256 tile. Tiles that reach past the matrix, shifts outside the
// conversions' window and the validation exports take the per-group path.
#pragma once
#include "call_header.h"
#include "gemm4_kernel.h"

namespace scalify {

__device__ __forceinline__ bool ge_fused(const GemmParams& p) {
  return p.res || p.act != ACT_NONE || p.ch_a || p.ch_b;
}

__device__ __forceinline__ void ge_store_f32(float* q, const v4f& v, int cols) {
  q[0] = v[0];
  if (cols > 1) q[1] = v[1];
  if (cols > 2) q[2] = v[2];
  if (cols > 3) q[3] = v[3];
}

// Decoded residual codes of columns n .. n + 3 of a residual that is one row
// for every row (a bias): the same for all of a thread's groups of a tile.
__device__ __forceinline__ v4f ge_bias(const GemmParams& p, int n) {
  v4f r = {0.f, 0.f, 0.f, 0.f};
  if (p.res && p.ldr == 0 && n < p.N) {
    uint32_t c[2];
    load_residual_codes(p, 0, n, c);
    r = p.res_fmt == kE4M3 ? decode_residual4(kE4M3, c[0], c[1])
                           : (p.res_fmt == kE5M2 ? decode_residual4(kE5M2, c[0], c[1])
                                                 : decode_residual4(kF16, c[0], c[1]));
  }
  return r;
}

// Residual codes of a batch, format RF (rows past the matrix: its last row,
// whose sums nobody uses). All loads of the batch are issued before the first
// is waited for.
template <int RF, int NB>
__device__ __forceinline__ void ge_load_residual(const GemmParams& p, int m, int dm, int n,
                                                 int cols, v4f (&r)[NB]) {
  uint32_t c[NB][2];
  if (cols >= 4) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int64_t e = (int64_t)min(m + j * dm, p.M - 1) * p.ldr + n;
      if constexpr (RF == kF16) {
        const v2i w = *(const v2i*)((const uint16_t*)p.res + e);
        c[j][0] = (uint32_t)w.x;
        c[j][1] = (uint32_t)w.y;
      } else {
        c[j][0] = *(const uint32_t*)((const uint8_t*)p.res + e);
        c[j][1] = 0u;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j) load_residual_codes(p, min(m + j * dm, p.M - 1), n, c[j]);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) r[j] = decode_residual4(RF, c[j][0], c[j][1]);
}

// v = fl(v * 2^(sh_acc + ch) + r * 2^sh_res), ch the channel exponents of the
// row (ea) and the columns (chb).
template <bool CH, int NB>
__device__ __forceinline__ void ge_add(v4f (&v)[NB], const v4f (&r)[NB], int sh_acc, int sh_res,
                                       const int (&ea)[NB], const int (&chb)[4]) {
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[j][i] = ldexpf(v[j][i], CH ? sh_acc + ea[j] + chb[i] : sh_acc) + ldexpf(r[j][i], sh_res);
}

// Activation X_d * g(X_d * X_s), the gate at the true value v * 2^e_w.
template <int ACT, int NB>
__device__ __forceinline__ void ge_activate(v4f (&v)[NB], int e_w) {
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = v[j][i];
      if constexpr (ACT == ACT_RELU) v[j][i] = x * (x > 0.0f ? 1.0f : 0.0f);
      else v[j][i] = x * smooth_gate<ACT == ACT_GELU_TANH>(ldexpf(x, e_w));
    }
}

// From accumulators to pre-cast values w of a batch (cols > 0 columns of the
// matrix): exports, channel scales, scaled add, activation.
template <int NB>
__device__ __forceinline__ void ge_values(const GemmParams& p, v4f (&v)[NB], int m, int dm, int n,
                                          int cols, const CallExponents& x, const v4f& bias) {
  if (p.acc_out) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (m + j * dm < p.M) ge_store_f32(p.acc_out + (int64_t)(m + j * dm) * p.N + n, v[j], cols);
  }
  const bool ch = p.ch_a || p.ch_b;
  int ea[NB], chb[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < NB; ++j) ea[j] = 0;
  if (ch) {
    if (p.ch_a) {
      float a[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) a[j] = p.ch_a[min(m + j * dm, p.M - 1)];
#pragma unroll
      for (int j = 0; j < NB; ++j) ea[j] = pow2_exponent_of(a[j]);
    }
    if (p.ch_b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) chb[i] = pow2_exponent_of(p.ch_b[min(n + i, p.N - 1)]);
    }
  }
  if (p.res) {
    v4f r[NB];
    if (p.ldr == 0) {
#pragma unroll
      for (int j = 0; j < NB; ++j) r[j] = bias;
    } else if (p.res_fmt == kE4M3) {
      ge_load_residual<kE4M3>(p, m, dm, n, cols, r);
    } else if (p.res_fmt == kE5M2) {
      ge_load_residual<kE5M2>(p, m, dm, n, cols, r);
    } else {
      ge_load_residual<kF16>(p, m, dm, n, cols, r);
    }
    if (ch) ge_add<true>(v, r, x.sh_acc, x.sh_res, ea, chb);
    else ge_add<false>(v, r, x.sh_acc, x.sh_res, ea, chb);
  } else if (ch) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j][i] = ldexpf(v[j][i], ea[j] + chb[i]);
  }
  if (p.act == ACT_RELU) ge_activate<ACT_RELU>(v, x.e_w);
  else if (p.act == ACT_GELU_TANH) ge_activate<ACT_GELU_TANH>(v, x.e_w);
  else if (p.act == ACT_SILU) ge_activate<ACT_SILU>(v, x.e_w);
  if (p.pre_out) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (m + j * dm < p.M) ge_store_f32(p.pre_out + (int64_t)(m + j * dm) * p.N + n, v[j], cols);
  }
}

// max |w| of a batch's outputs inside the matrix, into lmax (NaN ignored).
template <int NB>
__device__ __forceinline__ void ge_fold(const GemmParams& p, const v4f (&v)[NB], int m, int dm,
                                        int cols, bool inside, float& lmax) {
  if (inside) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      lmax = fmaxf(lmax, fmaxf(fmaxf(fabsf(v[j][0]), fabsf(v[j][1])),
                               fmaxf(fabsf(v[j][2]), fabsf(v[j][3]))));
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (m + j * dm < p.M) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < cols) lmax = fmaxf(lmax, fabsf(v[j][i]));
      }
  }
}

// How the call casts: its shift, and whether the conversions take it.
struct CastRule {
  int shift;
  bool fast, sat;
  float scale, inv;
};
__device__ __forceinline__ CastRule cast_rule(int shift, bool sat) {
  const bool fast = shift >= kFastShiftMinSub && shift <= kFastShiftMax;
  return CastRule{shift, fast, sat, fast ? pow2_float(shift) : 1.0f, fast ? pow2_float(-shift) : 1.0f};
}

// One group of 4 codes, any shift, any value, cols of them stored.
__device__ __forceinline__ void ge_store_codes1(const GemmParams& p, const v4f& v, int m, int n,
                                                int cols, const CastRule& c) {
  if (p.out_fmt == kF16) {
    const v2i w = cast4_f16_any(v, c.fast, c.inv, c.shift, c.sat);
    uint16_t* q = (uint16_t*)p.out + (int64_t)m * p.ldc + n;
    if (cols >= 4) {
      *(v2i*)q = w;
    } else {
      q[0] = (uint16_t)w.x;
      if (cols > 1) q[1] = (uint16_t)((uint32_t)w.x >> 16);
      if (cols > 2) q[2] = (uint16_t)w.y;
    }
  } else {
    const uint32_t w = p.out_fmt == kE4M3
                           ? cast4_fp8_any<kE4M3>(v, c.fast, c.scale, c.shift, c.sat)
                           : cast4_fp8_any<kE5M2>(v, c.fast, c.scale, c.shift, c.sat);
    uint8_t* q = (uint8_t*)p.out + (int64_t)m * p.ldc + n;
    if (cols >= 4) {
      *(uint32_t*)q = w;
    } else {
      q[0] = (uint8_t)w;
      if (cols > 1) q[1] = (uint8_t)(w >> 8);
      if (cols > 2) q[2] = (uint8_t)(w >> 16);
    }
  }
}

__device__ __forceinline__ bool ge_nan4(const v4f& v) {
  return v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3];
}

// A batch inside the matrix, the shift inside the conversions' window: the
// conversion scales by itself; a group that holds a NaN (rare) is patched.
template <int OF, bool SAT, int NB>
__device__ __forceinline__ void ge_store_codes_fast(const GemmParams& p, const v4f (&v)[NB], int m,
                                                    int dm, int n, const CastRule& c) {
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int64_t e = (int64_t)(m + j * dm) * p.ldc + n;
    if constexpr (OF == kF16) {
      v2i w = cvt4_f16_fast<SAT>(v[j][0], v[j][1], v[j][2], v[j][3], c.inv);
      if (__builtin_expect(ge_nan4(v[j]), 0)) w = cast4_f16_any(v[j], true, c.inv, c.shift, SAT);
      *(v2i*)((uint16_t*)p.out + e) = w;
    } else {
      uint32_t w = cast4_fp8_hw<OF>(__float_as_uint(v[j][0]), __float_as_uint(v[j][1]),
                                    __float_as_uint(v[j][2]), __float_as_uint(v[j][3]), c.scale, SAT);
      if (__builtin_expect(ge_nan4(v[j]), 0)) w = cast4_fp8_any<OF>(v[j], true, c.scale, c.shift, SAT);
      *(uint32_t*)((uint8_t*)p.out + e) = w;
    }
  }
}

template <int NB>
__device__ __forceinline__ void ge_store_codes(const GemmParams& p, const v4f (&v)[NB], int m,
                                               int dm, int n, int cols, bool inside,
                                               const CastRule& c) {
  if (inside && c.fast) {
    if (p.out_fmt == kE4M3)
      c.sat ? ge_store_codes_fast<kE4M3, true>(p, v, m, dm, n, c)
            : ge_store_codes_fast<kE4M3, false>(p, v, m, dm, n, c);
    else if (p.out_fmt == kE5M2)
      c.sat ? ge_store_codes_fast<kE5M2, true>(p, v, m, dm, n, c)
            : ge_store_codes_fast<kE5M2, false>(p, v, m, dm, n, c);
    else
      c.sat ? ge_store_codes_fast<kF16, true>(p, v, m, dm, n, c)
            : ge_store_codes_fast<kF16, false>(p, v, m, dm, n, c);
    return;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (m + j * dm < p.M) ge_store_codes1(p, v[j], m + j * dm, n, cols, c);
}

// The pre-cast intermediate of a batch (16-bit rounding-preserving encoding
// or fp32; its rows are padded to 16 elements, so whole groups are stored).
template <int NB>
__device__ __forceinline__ void ge_store_inter(const GemmParams& p, const v4f (&v)[NB], int m,
                                               int dm, int n) {
  if (p.epi == EPI_INTER16) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (m + j * dm >= p.M) continue;
      uint32_t x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t u = __float_as_uint(v[j][i]);
        x[i] = u | ((u & 0xFFFFu) + 0xFFFFu);  // sticky16(u) in bits 16..
      }
      *(v2i*)((uint16_t*)p.inter + (int64_t)(m + j * dm) * p.ldw + n) =
          v2i{(int)__builtin_amdgcn_perm(x[1], x[0], 0x07060302u),
              (int)__builtin_amdgcn_perm(x[3], x[2], 0x07060302u)};
    }
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (m + j * dm < p.M) *(v4f*)((float*)p.inter + (int64_t)(m + j * dm) * p.ldw + n) = v[j];
  }
}

// Cast of the whole intermediate by one workgroup (the recovery of the
// single pass when the grid was not co-resident).
__device__ __forceinline__ void ge_cast_all(const GemmParams& p, int tid, int threads,
                                            const CastRule& c) {
  const int gpr = (p.N + 3) / 4;
  for (int64_t g = tid; g < (int64_t)p.M * gpr; g += threads) {
    const int m = (int)(g / gpr), n = 4 * (int)(g % gpr);
    v4f v;
    if (p.epi == EPI_INTER16) {
      const v2i w = *(const v2i*)((const uint16_t*)p.inter + (int64_t)m * p.ldw + n);
      v = v4f{__uint_as_float((uint32_t)w.x << 16), __uint_as_float((uint32_t)w.x & 0xFFFF0000u),
              __uint_as_float((uint32_t)w.y << 16), __uint_as_float((uint32_t)w.y & 0xFFFF0000u)};
    } else {
      v = *(const v4f*)((const float*)p.inter + (int64_t)m * p.ldw + n);
    }
    ge_store_codes1(p, v, m, n, min(p.N - n, 4), c);
  }
}

}  // namespace scalify
