// Scaled FP8 GEMM for outputs that 256 x 256 tiles do not spread over the
// chip: the FP8 dot_general with fp32 accumulation of the scaled matmul
// (Section 3.2 / Algorithm 3) with every epilogue of the path but MX block
// scales.
//
// One workgroup of 4 waves (2 x 2) per 128 x TN tile, TN = 32 NI: each wave
// 64 x 16 NI outputs in 4 NI accumulator tiles. K in 128-byte steps through
// a ring of S LDS stages (buffer_load ... lds, range-checked).
//
// Main loop, one barrier per step, software pipelined by one step: wait for
// this wave's loads of step i + 1; barrier (the stage of step i has been read
// by everyone, step i + 1 has landed for everyone); then the MFMAs of step i
// from registers, and among them, one by one, the loads of step i + S into the
// freed stage and the LDS reads of step i + 1's fragments. Every wave's MFMAs, LDS reads and loads are spread evenly over
// the step, as the one wave of a SIMD cannot hide a burst of any of them.
//
// Epilogue: the accumulators go through LDS as one fp32 tile (it takes the
// stages' place), from which every thread takes groups of 4 consecutive
// outputs of a row; a wave covers whole row segments, so stores are coalesced
// and the code does not grow with the tile. In the single pass of the dynamic
// rescale (Section 3.3) the tile stays there across the grid barrier.
#pragma once
#include "mid_gemm.h"
#include "wave_gemm_kernel.h"

namespace scalify {

constexpr int MD_THREADS = 256;

// Byte of chunk `chunk` (16 bytes) of k-row k in an MC tile of W bytes per k-row.
template <int W>
__device__ __forceinline__ int md_swz(int k) {
  if constexpr (W == 256) return (k & 7) | (wv_kbit(k) << 3);
  else return ((k >> 1) & 3) | (wv_kbit(k) << 2);  // W = 128
}

// Read S of a fragment (KC: two 16-byte halves, MC: four transposing reads).
template <bool KC, int W, int S>
__device__ __forceinline__ void md_read_part(v8i& f, const uint8_t* lds, int base, int lane) {
  if constexpr (KC) {
    read_frag_part<true, S>(f, lds, base, lane);
  } else {
    const int t = lane & 15, g = lane >> 4;
    const int k = 32 * g + 8 * S + (t >> 1);
    const int off = k * W + 16 * ((base >> 4) ^ md_swz<W>(k)) + (t & 1) * 8;
    const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_AS v2i*)(lds + off));
    f[2 * S] = v.x;
    f[2 * S + 1] = v.y;
  }
}

// Offsets of a wave's LQ loads (1 KiB each) of an operand tile of R rows (KC)
// or R bytes per k-row (MC): a few per-lane parts, which differ by the chunk
// permutation, and a scalar part per load.
template <bool KC, int R, int LQ>
struct MidLoader {
  static constexpr int V = KC ? 2 : (R == 256 ? 4 : 2);  // different lane parts
  uint32_t lane_off[V];
  int kc[2];  // KC: k offset of the lane's chunk, per block parity

  static __device__ __forceinline__ constexpr int variant(int q) {
    return KC ? (q & 1) : (R == 256 ? (q & 1) + 2 * ((q >> 2) & 1) : ((q >> 1) & 1));
  }
  // k-rows (MC) or rows (KC) per load
  static constexpr int STEP = KC ? 8 : 1024 / R;

  __device__ __forceinline__ void init(uint32_t ld, int wave, int lane) {
#pragma unroll
    for (int par = 0; par < 2; ++par) kc[par] = 16 * ((lane & 7) ^ (lane >> 3) ^ par);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if constexpr (KC) {
        lane_off[v] = (uint32_t)(lane >> 3) * ld + (uint32_t)kc[v];
      } else {
        constexpr int CPR = R / 16;
        const int q = R == 256 ? (v & 1) + 4 * (v >> 1) : 2 * v;  // a load of this variant
        const int k = (wave * LQ + q) * STEP + lane / CPR;
        lane_off[v] = (uint32_t)(lane / CPR) * ld + 16u * (uint32_t)((lane % CPR) ^ md_swz<R>(k));
      }
    }
  }
  // Scalar part of load 0 of the tile at (row0, k0); load q is q * STEP * ld
  // further. Past K (ok false): out of range.
  static __device__ __forceinline__ uint32_t base(v4i rsrc, uint32_t ld, int row0, uint32_t k0,
                                                  bool ok, int wave) {
    const uint32_t first = (uint32_t)(wave * LQ * STEP);
    const uint32_t b = KC ? ((uint32_t)row0 + first) * ld + k0 : (k0 + first) * ld + (uint32_t)row0;
    return ok ? b : (uint32_t)rsrc.z;
  }
  __device__ __forceinline__ void issue(v4i rsrc, uint32_t base, uint32_t k0, int K, int wave, int q,
                                        uint8_t* lds) const {
    uint32_t o = lane_off[variant(q)] + base;
    if constexpr (KC) o = (int)k0 + kc[q & 1] >= K ? (uint32_t)rsrc.z : o;
    load_lds16(rsrc, o, lds + (wave * LQ + q) * 1024);
  }
};

template <bool A_MN, bool B_KC, int FA, int FB, int NI, int S>
__global__ __launch_bounds__(MD_THREADS, S == 2 ? 2 : 1) void mid_gemm_kernel(GemmParams p) {
  constexpr int MI = 4, TM = kMidTM, TN = 32 * NI;
  constexpr int ABYTES = TM * 128, BBYTES = TN * 128;
  constexpr int STAGE = ABYTES + BBYTES;
  constexpr int LA = 4, LB = NI;                         // loads per wave and step
  constexpr int LPS = LA + LB;
  constexpr int RLD = TN + 4;                            // row stride of the fp32 tile
  constexpr int TILE = TM * RLD * 4;
  constexpr int LDS = S * STAGE > TILE ? S * STAGE : TILE;
  constexpr int DSA = A_MN ? 4 : 2, DSB = B_KC ? 2 : 4;  // LDS reads per fragment
  constexpr int MF = MI * NI;                            // MFMAs per step
  constexpr bool PINNED = NI == 8;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
  __shared__ float red[4];
  __shared__ uint32_t sp_word[2];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = p.M, N = p.N, K = p.K;
  const int G = gridDim.x, T = p.tiles_m * p.tiles_n;
  const int KT = (K + BK - 1) / BK;
  const int KT_full = K / BK;
  const int krem = K - KT_full * BK;
  const uint32_t lda = (uint32_t)p.lda, ldb = (uint32_t)p.ldb;
  const v4i ra = make_rsrc(p.a, p.a_bytes);
  const v4i rb = make_rsrc(p.b, p.b_bytes);
  const int wm = 64 * (wave >> 1), wn = 16 * NI * (wave & 1);
  const RawScales raw_scales = load_scales(p);
  const bool first = blockIdx.x == 0 && tid == 0 && p.uses_header;
  const bool fuse = ge_fused(p);
  float* tile = (float*)lds;
  // this thread's groups of a tile: columns tcol .. + 3 of rows trow + DM j
  constexpr int GPR = TN / 4, DM = MD_THREADS / GPR, NB = 8, BATCHES = TM / (DM * NB);
  const int trow = tid / GPR, tcol = 4 * (tid % GPR);
  float lmax = 0.f;
  int m0, n0;

  for (int t = blockIdx.x; t < T; t += G) {
  wv_origin(t, p.tiles_m, p.tiles_n, TM, TN, m0, n0);
  // (recomputed for each tile: hoisted out of the tile loop, the per-lane
  // addresses of every fragment read would live in registers of their own)
  int lane = tid & 63;
  asm volatile("" : "+v"(lane));
  MidLoader<!A_MN, TM, LA> la;
  MidLoader<B_KC, TN, LB> lb;
  la.init(lda, wave, lane);
  lb.init(ldb, wave, lane);

  // Load j of step i (a step past K: zeros, no memory touched); the loads of
  // a step are issued in order, from the scalar offset that `begin` sets.
  uint32_t base_a, base_b;
  auto begin = [&](int i) {
    const uint32_t k0 = (uint32_t)i * BK;
    base_a = la.base(ra, lda, m0, k0, i < KT, wave);
    base_b = lb.base(rb, ldb, n0, k0, i < KT, wave);
  };
  auto issue_one = [&](int j, int i, uint8_t* st) {
    const uint32_t k0 = (uint32_t)i * BK;
    if (j < LA) {
      la.issue(ra, base_a, k0, K, wave, j, st);
      base_a += la.STEP * lda;
    } else {
      lb.issue(rb, base_b, k0, K, wave, j - LA, st + ABYTES);
      base_b += lb.STEP * ldb;
    }
  };

  // Fragments: A's of a step in one of two register sets; B's column groups
  // 0 .. NI - 3 in place (the next step's fragment is read into the registers
  // once the group's MFMAs have issued), the last two groups in two sets.
  v8i fa[2][MI], fb[NI + 2];
  constexpr int NP = NI - 2;  // column groups read in place
  // LDS read q of A's fragments / of B's group g for a step of parity P
  auto read_a = [&](auto Q, auto P, const uint8_t* st) {
    constexpr int q = decltype(Q)::value;
    md_read_part<!A_MN, TM, q % DSA>(fa[decltype(P)::value][q / DSA], st, wm + 16 * (q / DSA),
                                         lane);
  };
  auto read_b = [&](auto Gr, auto Q, auto P, const uint8_t* st) {
    constexpr int g = decltype(Gr)::value;
    md_read_part<B_KC, TN, decltype(Q)::value>(fb[g < NP ? g : g + 2 * decltype(P)::value],
                                                   st + ABYTES, wn + 16 * g, lane);
  };
  // The partial last step (step i of stage st), once landed: clear KC bytes >= K.
  auto zero_tail = [&](int i, uint8_t* st) {
    if (i == KT_full && (krem & 15)) {
      if (!A_MN && tid < TM) zero_tail_kc(st, krem, tid);
      if (B_KC && tid < TN) zero_tail_kc(st + ABYTES, krem, tid);
      __syncthreads();
    }
  };

  // NI = 8: the accumulators pinned in AGPRs (AccTile), as 128 of them rotate
  // through copies in the compiler's hands; NI = 4: ordinary values.
  v4f acc[PINNED ? 1 : MI][PINNED ? 1 : NI];
  static_for<0, MF>([&](auto I) {
    constexpr int t = decltype(I)::value;
    if constexpr (PINNED) AccTile<t>::zero();
    else acc[t / NI][t % NI] = v4f{0.f, 0.f, 0.f, 0.f};
  });

  if (KT > 0) {
    static_for<0, S - 1>([&](auto I) {
      begin(decltype(I)::value);
      for (int j = 0; j < LPS; ++j) issue_one(j, decltype(I)::value, lds + decltype(I)::value * STAGE);
    });
    bool opens = first && t == 0 && header_begin(p, raw_scales);
    wait_vmcnt<(S - 2) * LPS>();
    __syncthreads();
    zero_tail(0, lds);
    begin(S - 1);
    for (int j = 0; j < LPS; ++j) issue_one(j, S - 1, lds + (S - 1) * STAGE);
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    static_for<0, MI * DSA>([&](auto Q) { read_a(Q, P0{}, lds); });
    static_for<0, NI * DSB>([&](auto I) {
      constexpr int i = decltype(I)::value;
      read_b(std::integral_constant<int, i / DSB>{}, std::integral_constant<int, i % DSB>{}, P0{}, lds);
    });
    wait_lgkmcnt<0>();
    mfma_drain();  // (the zeroing, before the first MFMAs read it)
    __builtin_amdgcn_sched_barrier(0);
    int st_i = 0;  // stage of step i
    auto step = [&](auto P, int i) {
      constexpr int par = decltype(P)::value;
      using PN = std::integral_constant<int, 1 - par>;
      uint8_t* here = lds + st_i * STAGE;
      st_i = st_i + 1 == S ? 0 : st_i + 1;
      uint8_t* there = lds + st_i * STAGE;
      wait_vmcnt<(S - 2) * LPS>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      zero_tail(i + 1, there);
      begin(i + S);
      __builtin_amdgcn_sched_barrier(0);
      // MFMA m belongs to column group m / MI. Reads: those with registers of
      // their own (A, the last two B groups) evenly over the first RS MFMAs,
      // B group g over the MI MFMAs that follow its own.
      constexpr int RS = MF - MI;
      constexpr int FREE = MI * DSA + 2 * DSB;
      static_for<0, MF>([&](auto I) {
        constexpr int m = decltype(I)::value;
        constexpr int ni = m / MI, mi = m % MI;
        v8i& b = fb[ni < NP ? ni : ni + 2 * par];
        if constexpr (PINNED)
          AccTile<mi * NI + ni>::template mfma<FA, FB>(b, fa[par][mi]);
        else
          acc[mi][ni] = mfma<FA, FB>(b, fa[par][mi], acc[mi][ni]);
        if constexpr (m < RS) {
          static_for<m * FREE / RS, (m + 1) * FREE / RS>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            if constexpr (q < MI * DSA)
              read_a(Q, PN{}, there);
            else
              read_b(std::integral_constant<int, NP + (q - MI * DSA) / DSB>{},
                     std::integral_constant<int, (q - MI * DSA) % DSB>{}, PN{}, there);
          });
          if constexpr (ni >= 1 && ni - 1 < NP)
            static_for<mi * DSB / MI, (mi + 1) * DSB / MI>([&](auto Q) {
              read_b(std::integral_constant<int, ni - 1>{}, Q, PN{}, there);
            });
        }
        static_for<m * LPS / MF, (m + 1) * LPS / MF>([&](auto J) {
          issue_one(decltype(J)::value, i + S, here);
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      wait_lgkmcnt<0>();
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll 1
    for (int i = 0;;) {
      step(P0{}, i);
      if (opens) {
        wait_vmcnt<2 * LPS>();  // (its words, before the loads of two steps)
        header_publish(p);
        opens = false;
      }
      if (++i >= KT) break;
      step(P1{}, i);
      if (++i >= KT) break;
    }
    wait_vmcnt<0>();  // the zero loads past the last step
    mfma_drain();
  } else {
    if (first && t == 0) header_open(p, raw_scales);
  }
  __syncthreads();

  // ---- epilogue: the fp32 tile in LDS, groups of 4 outputs per thread; the
  // statistic of plain outputs straight from the accumulators
  const bool inside = m0 + TM <= M && n0 + TN <= N;
  static_for<0, MF>([&](auto I) {
    constexpr int mi = decltype(I)::value / NI, ni = decltype(I)::value % NI;
    v4f v;
    if constexpr (PINNED) v = AccTile<mi * NI + ni>::read();
    else v = acc[mi][ni];
    *(v4f*)(tile + (wm + 16 * mi + (lane & 15)) * RLD + wn + 16 * ni + 4 * (lane >> 4)) = v;
    if (inside) {
      lmax = fuse ? lmax
                  : fmaxf(lmax, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
    } else if (!fuse) {
      const int cols = m0 + wm + 16 * mi + (lane & 15) < M
                           ? N - (n0 + wn + 16 * ni + 4 * (lane >> 4)) : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) lmax = fmaxf(lmax, i < cols ? fabsf(v[i]) : 0.f);
    }
    __builtin_amdgcn_sched_barrier(0);  // (a few accumulators at a time)
  });
  __syncthreads();
  const int n = n0 + tcol, cols = min(N - n, 4);
  const bool values = fuse || p.acc_out || p.pre_out;
  if (cols > 0 && (!p.single_pass || values)) {
    const CallExponents ex = call_exponents(p, raw_scales);
    const CastRule c = cast_rule(ex.shift, p.sat != 0);
    const v4f bias = ge_bias(p, n);
#pragma unroll 1
    for (int b = 0; b < BATCHES; ++b) {
      const int row = trow + b * NB * DM;
      float* q = tile + row * RLD + tcol;
      v4f v[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) v[j] = *(const v4f*)(q + j * DM * RLD);
      if (values) ge_values(p, v, m0 + row, DM, n, cols, ex, bias);
      if (fuse) ge_fold(p, v, m0 + row, DM, cols, inside, lmax);
      if (p.epi == EPI_DIRECT) {
        ge_store_codes(p, v, m0 + row, DM, n, cols, inside, c);
      } else if (!p.single_pass) {
        ge_store_inter(p, v, m0 + row, DM, n);
      } else if (fuse) {  // (read back by this thread alone)
#pragma unroll
        for (int j = 0; j < NB; ++j) *(v4f*)(q + j * DM * RLD) = v[j];
      }
    }
  }
  if (!p.single_pass) __syncthreads();  // (before the next tile's loads)
  }  // tiles

  for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
  if ((tid & 63) == 0) red[wave] = lmax;
  __syncthreads();
  const float wmax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const CallExponents ex = call_exponents(p, raw_scales);
  if (p.epi == EPI_DIRECT) {
    if (tid == 0) direct_finish(p, wmax, G, ex);
    return;
  }
  if (!p.single_pass) {
    if (tid == 0) pair_finish(p, wmax, ex.e_w);
    return;
  }
  // Single pass (one tile per workgroup): the tile in LDS is cast with the
  // rescale of the whole output's statistic; after an abort (the grid was not
  // co-resident) every workgroup writes its tile to the intermediate and the
  // last one casts.
  if (tid == 0) grid_wait(p, grid_arrive(p, wmax, G, ex.e_w), sp_word);
  __syncthreads();
  uint32_t amax_raw = sp_word[1];
  const bool inside = m0 + TM <= M && n0 + TN <= N;
  const int n = n0 + tcol, cols = min(N - n, 4);
  auto each_batch = [&](auto&& f) {
    if (cols <= 0) return;
#pragma unroll 1
    for (int b = 0; b < BATCHES; ++b) {
      const int row = trow + b * NB * DM;
      v4f v[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) v[j] = *(const v4f*)(tile + (row + j * DM) * RLD + tcol);
      f(v, m0 + row);
    }
  };
  bool cast_all = false;
  if (sp_word[0] == SP_ABORTED) {
    each_batch([&](const v4f(&v)[NB], int m) { ge_store_inter(p, v, m, DM, n); });
    if (!last_writer(p, G, sp_word, amax_raw)) return;
    cast_all = true;
  }
  int e_out;
  const CastRule c = cast_rule(sp_shift(amax_raw, ex.e_w, p.e_cc, p.target, &e_out), p.sat != 0);
  if (tid == 0 && (blockIdx.x == 0 || cast_all)) {
    *p.out_scale = pow2_float(e_out);
    if (p.amax_out) *p.amax_out = __uint_as_float(amax_raw) * pow2_float(-p.e_cc);
  }
  if (cast_all)
    ge_cast_all(p, tid, MD_THREADS, c);
  else
    each_batch([&](const v4f(&v)[NB], int m) { ge_store_codes(p, v, m, DM, n, cols, inside, c); });
}

template <bool A_MN, bool B_KC, int NI, int S>
struct MidFamily {
  template <int FA, int FB>
  struct F {
    static hipError_t run(const GemmParams& p, hipStream_t s) {
      hipLaunchKernelGGL((mid_gemm_kernel<A_MN, B_KC, FA, FB, NI, S>),
                         dim3(p.grid), dim3(MD_THREADS), 0, s, p);
      return hipGetLastError();
    }
  };
};

}  // namespace scalify
