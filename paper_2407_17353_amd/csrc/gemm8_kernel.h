// Scaled FP8 GEMM, 8 waves, two per SIMD, one workgroup per 256 x 256 tile,
// each wave a 64 x 128 sub-tile with VGPR accumulators: for what the 4-wave
// kernel's registers cannot hold. That is the fused epilogue (scaled add of a
// residual, channel scales, activation), whose per-value arithmetic the second
// wave of a SIMD overlaps, on outputs of many tiles, and block scales of
// A stored [K][M] with B stored [K][N] (the weight gradient's layout: four
// transposing reads per fragment of both operands).
// B fragments are read two column groups ahead; one barrier per step, before
// its last quarter: by then every wave holds the B fragments it still needs,
// so after it the step's stage is free and takes the loads of step s + 2, and
// each wave refills its A fragments with those of step s + 1 as soon as their
// last MFMA has issued. Matrix cores bound it (2 M N K): 8192 cubed with an
// E4M3 residual, direct cast, 442 us, against 465 - 484 us on the 128-row
// kernel, whose smaller tile reads more per product.
#pragma once
#include "call_header.h"
#include "gemm4_kernel.h"

namespace scalify {

// Issue chunk load q (0 .. BPW - 1; 1 KiB per wave instruction) of this
// wave's share of one operand tile for the k-step starting at k0.
// Out-of-matrix rows (beyond M or N for KC, beyond K for MC) read zeros
// through the buffer range check; KC chunks that start at or beyond K are
// sent out of range too, and a chunk straddling K is trimmed by
// zero_tail_kc.
// ok = false (no tile left to load: the persistent kernel's last steps)
// sends the whole load out of range.
template <bool KC, int BPW>
__device__ __forceinline__ void issue_block(v4i rsrc, const TileLoader& L, uint32_t ld, int row0,
                                            int k0, int K, uint8_t* lds, int wave, int q,
                                            bool ok = true) {
  const int blk = wave * BPW + q;
  uint32_t off;
  if (KC) {
    off = (uint32_t)(row0 + blk * 8) * ld + (uint32_t)k0 + L.lane_off[q & 1];
    if (k0 + L.kchunk[q & 1] >= K) off = (uint32_t)rsrc.z;
  } else {
    off = (uint32_t)(k0 + blk * 4) * ld + (uint32_t)row0 + L.lane_off[q & 1];
  }
  if (!ok) off = (uint32_t)rsrc.z;
  load_lds16(rsrc, off, lds + blk * 1024);
}

static __device__ __attribute__((noinline)) v2i cast4_slow_f16(uint32_t u0, uint32_t u1, uint32_t u2,
                                                         uint32_t u3, int shift, bool sat) {
  return v2i{(int)(cast_bits<kF16>(u0, shift, sat) | (cast_bits<kF16>(u1, shift, sat) << 16)),
             (int)(cast_bits<kF16>(u2, shift, sat) | (cast_bits<kF16>(u3, shift, sat) << 16))};
}

static __device__ __attribute__((noinline)) uint32_t cast4_slow_fp8(int fmt, uint32_t u0, uint32_t u1,
                                                              uint32_t u2, uint32_t u3, int shift,
                                                              bool sat) {
  if (fmt == kE4M3)
    return cast_bits<kE4M3>(u0, shift, sat) | (cast_bits<kE4M3>(u1, shift, sat) << 8) |
           (cast_bits<kE4M3>(u2, shift, sat) << 16) | (cast_bits<kE4M3>(u3, shift, sat) << 24);
  return cast_bits<kE5M2>(u0, shift, sat) | (cast_bits<kE5M2>(u1, shift, sat) << 8) |
         (cast_bits<kE5M2>(u2, shift, sat) << 16) | (cast_bits<kE5M2>(u3, shift, sat) << 24);
}

// Channel exponents of a wave's outputs, packed 4 to a register as e + 128
// (channel scales lie in the E8M0 range [2^-127, 2^127]): cha[mi] for the
// row block (rows mb + 16 mi), chb[ni] byte i for column nb + 16 ni + i; 0
// where there is no channel scale or the output lies outside the matrix.
// All loads are issued before the first use; the packed form keeps the
// registers free for the residual codes loaded next.
template <int MI_, int NI_>
__device__ __forceinline__ void load_channel_exponents(const GemmParams& p, int mb, int nb,
                                                       int (&cha)[MI_], uint32_t (&chb)[NI_]) {
  float va[MI_];
  v4f vb[NI_];
#pragma unroll
  for (int mi = 0; mi < MI_; ++mi) {
    const int m = mb + 16 * mi;
    va[mi] = (p.ch_a && m < p.M) ? p.ch_a[m] : 1.0f;
  }
#pragma unroll
  for (int ni = 0; ni < NI_; ++ni) {
    const int n = nb + 16 * ni;
    if (p.ch_b && n + 3 < p.N) {
      vb[ni] = *(const v4f*)(p.ch_b + n);
    } else {
      vb[ni] = v4f{1.f, 1.f, 1.f, 1.f};
      if (p.ch_b) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < p.N) vb[ni][i] = p.ch_b[n + i];
      }
    }
  }
#pragma unroll
  for (int mi = 0; mi < MI_; ++mi) cha[mi] = pow2_exponent_of(va[mi]);
#pragma unroll
  for (int ni = 0; ni < NI_; ++ni) {
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) w |= (uint32_t)(pow2_exponent_of(vb[ni][i]) + 128) << (8 * i);
    chb[ni] = w;
  }
}

__device__ __forceinline__ int chb_exp(uint32_t packed, int i) {
  return (int)((packed >> (8 * i)) & 0xFFu) - 128;
}

template <int RF, bool CH, int MI_, int NI_>
__device__ __forceinline__ void add_residual(const GemmParams& p, v4f (&acc)[MI_][NI_], int mb,
                                             int nb, bool interior, int sh_acc, int sh_res,
                                             const int (&cha)[MI_], const uint32_t (&chb)[NI_]) {
  constexpr int W = RF == kF16 ? 2 : 1;  // code words per 4 outputs
  uint32_t rc[MI_][NI_][W];
  if (interior) {
    static_for<0, MI_ * NI_>([&](auto I) {
      constexpr int mi = decltype(I)::value / NI_, ni = decltype(I)::value % NI_;
      const int64_t e = (int64_t)(mb + 16 * mi) * p.ldr + nb + 16 * ni;
      if constexpr (RF == kF16) {
        const v2i w = *(const v2i*)((const uint16_t*)p.res + e);
        rc[mi][ni][0] = (uint32_t)w.x;
        rc[mi][ni][W - 1] = (uint32_t)w.y;
      } else {
        rc[mi][ni][0] = *(const uint32_t*)((const uint8_t*)p.res + e);
      }
    });
  } else {
    static_for<0, MI_ * NI_>([&](auto I) {
      constexpr int mi = decltype(I)::value / NI_, ni = decltype(I)::value % NI_;
      const int m = mb + 16 * mi;
      const int n = nb + 16 * ni;
      uint32_t c[2] = {0u, 0u};
      if (m < p.M && n < p.N) load_residual_codes(p, m, n, c);
      rc[mi][ni][0] = c[0];
      rc[mi][ni][W - 1] = RF == kF16 ? c[1] : c[0];
    });
  }
  static_for<0, MI_ * NI_>([&](auto I) {
    constexpr int mi = decltype(I)::value / NI_, ni = decltype(I)::value % NI_;
    const v4f r = decode_residual4(RF, rc[mi][ni][0], rc[mi][ni][W - 1]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc[mi][ni][i] = ldexpf(acc[mi][ni][i], CH ? sh_acc + cha[mi] + chb_exp(chb[ni], i) : sh_acc) +
                       ldexpf(r[i], sh_res);
    __builtin_amdgcn_sched_barrier(0);  // one group at a time: bounded register use
  });
}

template <int ACT, int MI_, int NI_>
__device__ __forceinline__ void activate(v4f (&acc)[MI_][NI_], int e_w) {
  static_for<0, MI_ * NI_>([&](auto I) {
    constexpr int mi = decltype(I)::value / NI_, ni = decltype(I)::value % NI_;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = acc[mi][ni][i];
      if constexpr (ACT == ACT_RELU) {
        acc[mi][ni][i] = v * (v > 0.0f ? 1.0f : 0.0f);
      } else {
        acc[mi][ni][i] = v * smooth_gate<ACT == ACT_GELU_TANH>(ldexpf(v, e_w));
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // one group at a time: bounded register use
  });
}

// CH: the fused epilogue also applies channel scales (instantiated apart, so
// that the other fused kernels keep their register allocation).
template <bool A_MN, bool B_KC, int FA, int FB, int EPI, bool CH, bool MX>
__global__ __launch_bounds__(512, 1) void gemm8_kernel(GemmParams p) {
  static_assert(EPI == EPI_INTER32 || EPI == EPI_DIRECT, "fp32 intermediate or direct cast");
  static_assert(!MX || !CH, "block scales: plain epilogue");
  constexpr bool FUSE = !MX;
  using C = WaveCfg<8>;
  constexpr int WAVES = C::WAVES, WAVES_N = C::WAVES_N, WTM = C::WTM, WTN = C::WTN;
  constexpr int MI = C::MI, NI = C::NI, BPW = C::BPW, LOADS_PER_STEP = C::LOADS_PER_STEP;
  __shared__ __attribute__((aligned(1024))) uint8_t sA0[TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) uint8_t sB0[TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) uint8_t sA1[TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) uint8_t sB1[TILE_BYTES];
  __shared__ float red[WAVES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  int m0, n0;
  tile_origin(blockIdx.x, p.tiles_m, p.tiles_n, m0, n0);
  const RawScales raw_scales = load_scales(p);
  const bool first = blockIdx.x == 0 && tid == 0 && p.uses_header;

  const int M = p.M, N = p.N, K = p.K;
  const int KT = (K + BK - 1) / BK;
  const int KT_full = K / BK;         // k-steps entirely inside K
  const int krem = K - KT_full * BK;  // bytes of the partial last step (0 if none)
  const uint32_t lda = (uint32_t)p.lda, ldb = (uint32_t)p.ldb;

  // A: KC when stored [M][K], MC when stored [K][M] (row0 = m0 either way).
  // B: KC when stored [N][K], MC when stored [K][N].
  const v4i ra = make_rsrc(p.a, p.a_bytes);
  const v4i rb = make_rsrc(p.b, p.b_bytes);
  const TileLoader la = make_loader<!A_MN, BPW>(lda, wave, lane);
  const TileLoader lb = make_loader<B_KC, BPW>(ldb, wave, lane);

  // Load j of a step: j < BPW are A blocks, the rest B blocks.
  auto issue_one = [&](int j, int kt, uint8_t* dA, uint8_t* dB) {
    if (j < BPW)
      issue_block<!A_MN, BPW>(ra, la, lda, m0, kt * BK, K, dA, wave, j);
    else
      issue_block<B_KC, BPW>(rb, lb, ldb, n0, kt * BK, K, dB, wave, j - BPW);
  };
  auto issue_all = [&](int kt, uint8_t* dA, uint8_t* dB) {
#pragma unroll
    for (int j = 0; j < LOADS_PER_STEP; ++j) issue_one(j, kt, dA, dB);
  };
  // The partial last step's stage, once landed: clear the KC bytes >= K.
  auto zero_tail = [&](uint8_t* dA, uint8_t* dB) {
    if (!A_MN) zero_tail_kc(dA, krem, tid);
    if (B_KC) zero_tail_kc(dB, krem, tid);
    __syncthreads();
  };

  // MX block scales, packed (see GemmParams): a k-step's 256 bytes of one
  // 64-row group are contiguous, so wave w < 4 stages A's group m0 / 64 + w
  // and wave w >= 4 B's group n0 / 64 + w - 4 with one 256-byte load beside
  // the step's tiles (groups past the array read zeros: rows past M or N,
  // whose data are zero). Stage layout: [2 k-step stages][A 1 KiB | B 1 KiB],
  // tile group j at 256 j. Lane l's word of a group holds the bytes of its
  // 4 row blocks (rows l & 15, + 16, + 32, + 48) at k-block l >> 4.
  uint8_t* sS = nullptr;
  if constexpr (MX) {
    __shared__ __attribute__((aligned(1024))) uint8_t s_mx[4096];
    sS = s_mx;
  }
  auto issue_scales = [&](int kt, int stage) {
    if constexpr (MX) {
      const bool is_b = wave >= 4;
      const int groups = is_b ? p.mx_groups_b : p.mx_groups_a;
      const int grp = (is_b ? n0 : m0) / 64 + (wave & 3);
      const v4i r = is_b ? make_rsrc(p.mx_b, p.mx_b_bytes) : make_rsrc(p.mx_a, p.mx_a_bytes);
      const uint32_t off =
          grp < groups ? ((uint32_t)(kt * groups + grp) * 64u + (uint32_t)lane) * 4u : (uint32_t)r.z;
      load_lds4<0>(r, off, sS + stage * 2048 + (is_b ? 1024 : 0) + 256 * (wave & 3));
    }
  };
  // This lane's word of tile group j (0..3) of operand half (0 A, 1 B).
  auto scale_word = [&](int stage, int half, int j) -> int {
    return *(const int*)(sS + stage * 2048 + half * 1024 + 256 * j + 4 * lane);
  };

  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  const int wm = (wave / WAVES_N) * WTM;  // wave sub-tile
  const int wn = (wave % WAVES_N) * WTN;
  constexpr int DSA = A_MN ? 4 : 2;  // LDS reads per A fragment
  constexpr int DSB = B_KC ? 2 : 4;  // LDS reads per B fragment
  static_assert(LOADS_PER_STEP == 2 * MI, "two loads per row block");
  using T_ = std::true_type;
  using F_ = std::false_type;

  {
    v8i a[MI];   // A fragments of the step
    v8i bq[3];   // B fragments: in use and up to two groups ahead
    // MX: this lane's block-scale words of the step: A's for the wave's 64
    // rows (byte mi), B's for its column groups 0 .. 3 and 4 .. 7 (byte ni & 3)
    int sa = 0, sb[2] = {0, 0};
    static_assert(!MX || (MI == 4 && NI == 8 && WTM == 64 && WTN == 128), "MX word layout");

    // One k-step. LOADS: issue the loads of step kt + 2 into this step's
    // stage after the barrier. NEXT: step kt + 1 exists (barrier, then its A
    // fragments and first B fragment are read into a[] and b).
    auto step = [&](auto loads_tag, auto next_tag, int kt) {
      constexpr bool LOADS = decltype(loads_tag)::value;
      constexpr bool NEXT = decltype(next_tag)::value;
      const bool odd = kt & 1;
      uint8_t* cA = odd ? sA1 : sA0;  // this step's stage
      uint8_t* cB = odd ? sB1 : sB0;
      uint8_t* nA = odd ? sA0 : sA1;  // the next step's stage
      uint8_t* nB = odd ? sB0 : sB1;
      // B column groups 0 .. NI - 3, fragments read two groups ahead
      static_for<0, NI - 2>([&](auto I) {
        constexpr int ni = decltype(I)::value;
        bq[(ni + 2) % 3] = read_frag<B_KC, MX>(cB, wn + 16 * (ni + 2), lane);
        static_for<0, MI>([&](auto J) {
          constexpr int mi = decltype(J)::value;
          acc[mi][ni] =
              mfma_s<FA, FB, MX, ni & 3, mi>(bq[ni % 3], a[mi], acc[mi][ni], sb[ni >> 2], sa);
        });
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (mi < DSB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      });
      if (NEXT) {
        // Every wave holds all B fragments of this step once its LDS reads
        // have returned (the barrier waits for them), so this stage is free
        // after the barrier; step kt + 1 has landed once every wave's loads
        // have completed.
        wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        if (!LOADS && kt + 1 == KT_full && (krem & 15)) zero_tail(nA, nB);
        // MX: B column groups 0 .. 3 are done with their word
        if constexpr (MX) sb[0] = scale_word(!odd, 1, wn / 64);
      }
      // B column groups NI - 2 and NI - 1, taken row block by row block: once
      // both MFMAs of a[mi] have issued, a[mi] is refilled with the fragment
      // of step kt + 1; the loads of step kt + 2 go out two per row block.
      static_for<0, MI>([&](auto J) {
        constexpr int mi = decltype(J)::value;
        acc[mi][NI - 2] = mfma_s<FA, FB, MX, (NI - 2) & 3, mi>(bq[(NI - 2) % 3], a[mi],
                                                                acc[mi][NI - 2], sb[1], sa);
        acc[mi][NI - 1] = mfma_s<FA, FB, MX, (NI - 1) & 3, mi>(bq[(NI - 1) % 3], a[mi],
                                                                acc[mi][NI - 1], sb[1], sa);
        if (LOADS) {
          issue_one(2 * mi, kt + 2, cA, cB);
          issue_one(2 * mi + 1, kt + 2, cA, cB);
          if (mi == MI - 1) issue_scales(kt + 2, odd);
        }
        if (NEXT) a[mi] = read_frag<!A_MN, MX>(nA, wm + 16 * mi, lane);
      });
      if (NEXT) {
        bq[0] = read_frag<B_KC, MX>(nB, wn, lane);
        bq[1] = read_frag<B_KC, MX>(nB, wn + 16, lane);
        if constexpr (MX) {  // every MFMA of this step has issued
          sb[1] = scale_word(!odd, 1, wn / 64 + 1);
          sa = scale_word(!odd, 0, wm / 64);
        }
      }
      static_for<0, MI>([&](auto I) {
        constexpr int i = decltype(I)::value;
        // MX: one B word after the barrier, a B and the A word at the end
        constexpr int XS = MX ? (i == 0 ? 1 : 0) + (i + 1 == MI ? 2 : 0) : 0;
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        if (NEXT)
          __builtin_amdgcn_sched_group_barrier(0x100, (i + 1 < MI ? DSA : DSA + 2 * DSB) + XS, 0);
      });
    };

    if (KT > 0) {
      issue_all(0, sA0, sB0);
      issue_scales(0, 0);
      if (KT > 1) {
        issue_all(1, sA1, sB1);
        issue_scales(1, 1);
      }
      const bool opens = first && header_begin(p, raw_scales);
      if (KT > 1) {
        wait_vmcnt<LOADS_PER_STEP + (MX ? 1 : 0)>();  // step 1's loads may be in flight
      } else {
        wait_vmcnt<0>();
      }
      __syncthreads();
      if (KT_full == 0 && (krem & 15)) zero_tail(sA0, sB0);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) a[mi] = read_frag<!A_MN, MX>(sA0, wm + 16 * mi, lane);
      bq[0] = read_frag<B_KC, MX>(sB0, wn, lane);
      bq[1] = read_frag<B_KC, MX>(sB0, wn + 16, lane);
      if constexpr (MX) {
        sa = scale_word(0, 0, wm / 64);
        sb[0] = scale_word(0, 1, wn / 64);
        sb[1] = scale_word(0, 1, wn / 64 + 1);
      }
      if (opens) {
        wait_vmcnt<0>();  // (its words; the loads before them have landed)
        header_publish(p);
      }
    } else if (first) {
      header_open(p, raw_scales);
    }
    int kt = 0;
    for (; kt + 2 < KT; ++kt) step(T_{}, T_{}, kt);
    if (kt + 1 < KT) step(F_{}, T_{}, kt++);
    if (kt < KT) step(F_{}, F_{}, kt);
  }

  // ---- epilogue: lane holds C[m][n..n+3] for each (mi, ni)
  float lmax = 0.f;
  const int mb = m0 + wm + (lane & 15);
  const int nb = n0 + wn + 4 * (lane >> 4);
  const CallExponents ex = call_exponents(p, raw_scales);
  const int shift = ex.shift;  // EPI_DIRECT: data' = w * 2^-shift
  // (fused values and block-scaled accumulators may be fp32 subnormals)
  const bool fast = shift >= kFastShiftMinSub && shift <= kFastShiftMax;
  const float hw_scale = fast ? pow2_float(shift) : 1.0f;
  const float hw_inv = fast ? pow2_float(-shift) : 1.0f;
  const bool sat = p.sat != 0;
  // FUSE: a first pass turns every accumulator into its pre-cast value w
  // (scaled add, activation) before any store is issued, so that the only
  // memory waits are those of the residual codes, all loaded up front; the
  // pass below then writes w as the plain epilogue writes acc.
  if constexpr (FUSE) {
    if (p.acc_out) {
      static_for<0, MI * NI>([&](auto I) {
        constexpr int mi = decltype(I)::value / NI, ni = decltype(I)::value % NI;
        const int m = mb + 16 * mi;
        const int n = nb + 16 * ni;
        if (m < M && n < N) {
          const v4f a = acc[mi][ni];
          float* q = p.acc_out + (int64_t)m * N + n;
          q[0] = a[0];
          if (n + 1 < N) q[1] = a[1];
          if (n + 2 < N) q[2] = a[2];
          if (n + 3 < N) q[3] = a[3];
        }
      });
    }
    // Channel scales (CH): one power-of-two product of the accumulator,
    // folded into the scaled add's shift when there is a residual.
    int cha[MI] = {};
    uint32_t chb[NI] = {};
    if constexpr (CH) {
      load_channel_exponents(p, mb, nb, cha, chb);
      __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) chb[ni] = 0x80808080u;  // exponent 0
    }
    if (p.res) {
      const bool interior = m0 + wm + 16 * MI <= M && n0 + wn + 16 * NI <= N;
      const int sh_acc = ex.sh_acc, sh_res = ex.sh_res;
      if (p.res_fmt == kE4M3) add_residual<kE4M3, CH>(p, acc, mb, nb, interior, sh_acc, sh_res, cha, chb);
      else if (p.res_fmt == kE5M2) add_residual<kE5M2, CH>(p, acc, mb, nb, interior, sh_acc, sh_res, cha, chb);
      else add_residual<kF16, CH>(p, acc, mb, nb, interior, sh_acc, sh_res, cha, chb);
    } else if constexpr (CH) {
      static_for<0, MI * NI>([&](auto I) {
        constexpr int mi = decltype(I)::value / NI, ni = decltype(I)::value % NI;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[mi][ni][i] = ldexpf(acc[mi][ni][i], cha[mi] + chb_exp(chb[ni], i));
      });
    }
    if (p.act == ACT_RELU) activate<ACT_RELU>(acc, ex.e_w);
    else if (p.act == ACT_GELU_TANH) activate<ACT_GELU_TANH>(acc, ex.e_w);
    else if (p.act == ACT_SILU) activate<ACT_SILU>(acc, ex.e_w);
  }
  static_for<0, MI * NI>([&](auto I) {
    constexpr int mi = decltype(I)::value / NI, ni = decltype(I)::value % NI;
    const int m = mb + 16 * mi;
    const int n = nb + 16 * ni;
    if (m < M && n < N) {
      const v4f v = acc[mi][ni];  // FUSE: w
      lmax = fmaxf(lmax, fabsf(v[0]));
      if (n + 1 < N) lmax = fmaxf(lmax, fabsf(v[1]));
      if (n + 2 < N) lmax = fmaxf(lmax, fabsf(v[2]));
      if (n + 3 < N) lmax = fmaxf(lmax, fabsf(v[3]));
      if (EPI == EPI_INTER32) {
        float* q = (float*)p.inter + (int64_t)m * p.ldw + n;
        *(v4f*)q = v;
      } else {
        const uint32_t u0 = __float_as_uint(v[0]), u1 = __float_as_uint(v[1]);
        const uint32_t u2 = __float_as_uint(v[2]), u3 = __float_as_uint(v[3]);
        // Hardware conversions unless a lane of the wave holds a NaN or the
        // shift is out of their range (then the exact integer cast, out of
        // line: it is rare and large).
        const bool nan = is_nan_bits(u0) || is_nan_bits(u1) || is_nan_bits(u2) || is_nan_bits(u3);
        const bool hw = fast && !__any(nan);
        if (p.out_fmt == kF16) {
          v2i w;
          if (hw) {
            w = cast4_f16_hw(u0, u1, u2, u3, hw_inv, sat);
          } else {
            w = cast4_slow_f16(u0, u1, u2, u3, shift, sat);
          }
          uint16_t* q = (uint16_t*)p.out + (int64_t)m * p.ldc + n;
          if (n + 3 < N) {
            *(v2i*)q = w;
          } else {
            q[0] = (uint16_t)w.x;
            if (n + 1 < N) q[1] = (uint16_t)((uint32_t)w.x >> 16);
            if (n + 2 < N) q[2] = (uint16_t)w.y;
          }
        } else {
          uint32_t w;
          if (hw) {
            w = p.out_fmt == kE4M3 ? cast4_fp8_hw<kE4M3>(u0, u1, u2, u3, hw_scale, sat)
                                   : cast4_fp8_hw<kE5M2>(u0, u1, u2, u3, hw_scale, sat);
          } else {
            w = cast4_slow_fp8(p.out_fmt, u0, u1, u2, u3, shift, sat);
          }
          uint8_t* q = (uint8_t*)p.out + (int64_t)m * p.ldc + n;
          if (n + 3 < N) {
            *(uint32_t*)q = w;
          } else {
            q[0] = (uint8_t)w;
            if (n + 1 < N) q[1] = (uint8_t)(w >> 8);
            if (n + 2 < N) q[2] = (uint8_t)(w >> 16);
          }
        }
      }
      if (!FUSE && p.acc_out) {
        const v4f a = v;
        float* q = p.acc_out + (int64_t)m * N + n;
        q[0] = a[0];
        if (n + 1 < N) q[1] = a[1];
        if (n + 2 < N) q[2] = a[2];
        if (n + 3 < N) q[3] = a[3];
      }
      if constexpr (FUSE) {
        if (p.pre_out) {
          float* q = p.pre_out + (int64_t)m * N + n;
          q[0] = v[0];
          if (n + 1 < N) q[1] = v[1];
          if (n + 2 < N) q[2] = v[2];
          if (n + 3 < N) q[3] = v[3];
        }
      }
    }
  });
  // amax of |acc| over the valid elements (fmaxf ignores NaN): wave
  // butterfly, then across the waves, then one atomic max per workgroup
  // on the fp32 bits (non-negative floats order like their bits).
  for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
  if (lane == 0) red[wave] = lmax;
  __syncthreads();
  if (tid == 0) {
    float wmax = red[0];
    for (int w = 1; w < WAVES; ++w) wmax = fmaxf(wmax, red[w]);
    if (EPI == EPI_DIRECT) direct_finish(p, wmax, gridDim.x, ex);
    else pair_finish(p, wmax, ex.e_w);
  }
}

template <bool A_MN, bool B_KC>
struct FusedFamily {
  template <int FA, int FB>
  struct F {
    static hipError_t run(const GemmParams& p, hipStream_t s) {
      const bool ch = p.ch_a || p.ch_b;
      const dim3 g(p.tiles_m * p.tiles_n), b(512);
      if (p.epi == EPI_DIRECT) {
        if (ch) hipLaunchKernelGGL((gemm8_kernel<A_MN, B_KC, FA, FB, EPI_DIRECT, true, false>), g, b, 0, s, p);
        else hipLaunchKernelGGL((gemm8_kernel<A_MN, B_KC, FA, FB, EPI_DIRECT, false, false>), g, b, 0, s, p);
      } else {
        if (ch) hipLaunchKernelGGL((gemm8_kernel<A_MN, B_KC, FA, FB, EPI_INTER32, true, false>), g, b, 0, s, p);
        else hipLaunchKernelGGL((gemm8_kernel<A_MN, B_KC, FA, FB, EPI_INTER32, false, false>), g, b, 0, s, p);
      }
      return hipGetLastError();
    }
  };
};

}  // namespace scalify
