// Scaled FP8 GEMM for outputs of few 256 x 256 tiles (decode and other short
// batches, small squares): the FP8 dot_general with fp32 accumulation of the
// scaled matmul (Section 3.2 / Algorithm 3) with every epilogue of the path
// (dynamic, delayed or no rescale; scaled add, activation, channel scales;
// MX block scales).
//
// What bounds it: with 256 x 256 tiles such an output gives work to a few of
// the 256 CUs, each a serial chain of K / 128 steps (32 x 12288 x 4096: 48
// workgroups, 6 % of the tile rows real). Here the output is cut into TM x 64
// tiles (TM = 16, 32 or 64, the smallest that holds M), and K inside the
// workgroup: wave w of 4 takes the k-steps w, w + 4, ..., so that
//   * the chain of a wave is a quarter as long, and 4 waves stream operands
//     at once: 120 .. 150 KiB of loads in flight per CU;
//   * a wave's fragments come from LDS slots of its own: no barrier in the
//     main loop, only waits on its own loads (a ring of S slots per wave).
// The 4 partial tiles are summed through LDS in a fixed order (bit-identical
// reruns), which leaves each thread with groups of 4 consecutive outputs of
// a row; the epilogue works on those groups.
//
// Main loop of a wave, software pipelined by one step: wait for step i + 1's
// loads; read its fragments into the other register set; the MFMAs of step
// i; then refill the slot just read with step i + 1 + S. Steps past the end
// load zeros without touching memory (range-checked buffer loads), so the
// number of loads in flight is always known.
#pragma once
#include "group_epilogue.h"
#include "wave_gemm.h"

namespace scalify {

constexpr int WV_K = 4;       // waves, each a share of K
constexpr int WV_THREADS = 64 * WV_K;

// LDS tile of an operand stored along M or N ("MC"): W bytes per k-row. Chunk
// slots of 16 bytes are permuted so that the 16 rows which two neighbouring
// 16-lane groups read with one transposing load fall on distinct banks (for
// W = 16, one chunk per row, rows 8 apart trade places instead).
__device__ __forceinline__ int wv_kbit(int k) { return ((k >> 4) ^ (k >> 5)) & 1; }

template <int W>
__device__ __forceinline__ int wv_mc_off(int k, int chunk) {
  if constexpr (W == 64) return k * 64 + 16 * (chunk ^ ((((k >> 2) & 1)) | (wv_kbit(k) << 1)));
  else if constexpr (W == 32) return k * 32 + 16 * (chunk ^ wv_kbit(k));
  else return (k ^ (wv_kbit(k) << 3)) * 16;
}

// Offsets of an operand tile's loads (1 KiB each, R / 8 of them): rows (KC,
// 128 bytes along K) or k-rows (MC, R bytes along M / N), with the chunk
// permutation applied on the global side. The per-lane parts differ by the
// permutation only; the rest is a scalar per load.
template <bool KC, int R>
struct WaveLoader {
  static constexpr int Q = R / 8;
  static constexpr int STEP = KC ? 8 : 1024 / R;  // rows (k-rows) per load
  static constexpr int V = R == 16 && !KC ? 1 : 2;
  uint32_t lane_off[V];
  int kc[2];

  static __device__ __forceinline__ constexpr int variant(int q) {
    // KC: parity of the 8-row block; MC: bit 4 ^ bit 5 of the k-row (R = 64:
    // 16 k-rows per load, R = 32: 32, with bit 4 in the lane part)
    return KC ? (q & 1) : (R == 64 ? (q ^ (q >> 1)) & 1 : (R == 32 ? q & 1 : 0));
  }
  __device__ __forceinline__ void init(uint32_t ld, int lane) {
#pragma unroll
    for (int par = 0; par < 2; ++par) kc[par] = 16 * ((lane & 7) ^ (lane >> 3) ^ par);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if constexpr (KC) {
        lane_off[v] = (uint32_t)(lane >> 3) * ld + (uint32_t)kc[v];
      } else if constexpr (R == 16) {
        // 64 k-rows per load, the two halves of 16 rows swapped where the bit is set
        const int k = lane ^ (wv_kbit(lane) << 3);
        lane_off[v] = (uint32_t)k * ld;
      } else {
        constexpr int CPR = R / 16;
        const int k = v * STEP + lane / CPR, slot = lane % CPR;  // load v is of variant v
        const int c = R == 64 ? slot ^ (((k >> 2) & 1) | (wv_kbit(k) << 1)) : slot ^ wv_kbit(k);
        lane_off[v] = (uint32_t)(lane / CPR) * ld + (uint32_t)(16 * c);
      }
    }
  }
  // The loads of k-step kt (ok: it exists) of the tile at row0, into lds.
  __device__ __forceinline__ void issue(v4i rsrc, uint32_t ld, int row0, int kt, int K, bool ok,
                                        uint8_t* lds) const {
    const uint32_t k0 = (uint32_t)kt * BK;
    uint32_t base = KC ? (uint32_t)row0 * ld + k0 : k0 * ld + (uint32_t)row0;
    base = ok ? base : (uint32_t)rsrc.z;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t o = lane_off[variant(q)] + base;
      if constexpr (KC) o = (int)k0 + kc[q & 1] >= K ? (uint32_t)rsrc.z : o;
      load_lds16(rsrc, o, lds + q * 1024);
      base += (uint32_t)STEP * ld;
    }
  }
};

template <bool KC, int R, bool HWK>
__device__ __forceinline__ v8i wv_read_frag(const uint8_t* lds, int base, int lane) {
  if constexpr (KC) {
    return read_frag<true, HWK>(lds, base, lane);
  } else {
    v8i f;
    const int t = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = (HWK ? 64 * (s >> 1) + 16 * g + 8 * (s & 1) : 32 * g + 8 * s) + (t >> 1);
      const int off = wv_mc_off<R>(k, base >> 4) + (t & 1) * 8;
      const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_AS v2i*)(lds + off));
      f[2 * s] = v.x;
      f[2 * s + 1] = v.y;
    }
    return f;
  }
}

// KC tile of R rows: clear the bytes k >= krem of the chunk that straddles K.
template <int R>
__device__ __forceinline__ void wv_zero_tail(uint8_t* lds, int krem, int lane) {
  if (lane < R) {
    uint8_t* chunk = lds + lane * 128 + (((krem >> 4) ^ swz_kc(lane)) * 16);
    for (int b = krem & 15; b < 16; ++b) chunk[b] = 0;
  }
}

// Tile t of T, m fastest in groups of 8 tile rows: each XCD (workgroups are
// dealt over the 8 XCDs round robin) gets a contiguous range of tiles, for
// any T, so the tiles that run together on one share their panels in its L2.
__device__ __forceinline__ void wv_origin(int t, int tiles_m, int tiles_n, int tm, int tn, int& m0,
                                          int& n0) {
  const int T = tiles_m * tiles_n;
  const int x = t & 7, r = T & 7;
  t = x * (T >> 3) + (x < r ? x : r) + (t >> 3);
  constexpr int G = 8;
  const int group = t / (G * tiles_n);
  const int first_m = group * G;
  const int gm = min(tiles_m - first_m, G);
  const int in_group = t - group * G * tiles_n;
  m0 = (first_m + in_group % gm) * tm;
  n0 = (in_group / gm) * tn;
}

// MI: rows of the tile / 16 (1, 2 or 4); the tile is 16 MI x 64.
template <bool A_MN, bool B_KC, int FA, int FB, bool MX, int MI>
__global__ __launch_bounds__(WV_THREADS, 1) void wave_gemm_kernel(GemmParams p) {
  constexpr int NI = kWaveTN / 16, TM = 16 * MI, TN = kWaveTN;
  constexpr int ABYTES = TM * 128, BBYTES = TN * 128;
  constexpr int SLOT = ABYTES + BBYTES + (MX ? 512 : 0);
  constexpr int S = MI == 4 ? 2 : 3;                    // slots of a wave's ring
  constexpr int LPS = TM / 8 + TN / 8 + (MX ? 2 : 0);   // loads per step
  static_assert((S - 1) * LPS < 64 && 2 * LPS < 64, "vmcnt range");
  constexpr int RLD = TN + 4;                           // row stride of the partial tiles (floats)
  static_assert(4 * TM * RLD * 4 <= 4 * S * SLOT, "partial tiles fit the ring");
  constexpr int NG = MI;                                // groups of 4 outputs per thread
  static_assert(TN == 64 && WV_THREADS == 256, "16 groups per row: thread rows 16 apart");
  __shared__ __attribute__((aligned(1024))) uint8_t ring[WV_K * S * SLOT];
  __shared__ float red[WV_K];
  __shared__ uint32_t sp_word[2];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = p.M, N = p.N, K = p.K;
  const int G = gridDim.x;
  const int T = p.tiles_m * p.tiles_n;
  const int KT = (K + BK - 1) / BK;
  const int KT_full = K / BK;
  const int krem = K - KT_full * BK;
  const int steps = (KT - wave + WV_K - 1) / WV_K;      // of this wave (0 or more)
  const uint32_t lda = (uint32_t)p.lda, ldb = (uint32_t)p.ldb;
  const v4i ra = make_rsrc(p.a, p.a_bytes);
  const v4i rb = make_rsrc(p.b, p.b_bytes);
  uint8_t* mine = ring + wave * (S * SLOT);

  const RawScales raw_scales = load_scales(p);
  const bool first = blockIdx.x == 0 && tid == 0 && p.uses_header;
  const bool fuse = ge_fused(p);
  const int trow = tid >> 4, tcol = 4 * (tid & 15);     // this thread's groups in a tile
  float lmax = 0.f;
  v4f held[kWaveHeld][NG];
#pragma unroll
  for (int h = 0; h < kWaveHeld; ++h)
#pragma unroll
    for (int j = 0; j < NG; ++j) held[h][j] = v4f{0.f, 0.f, 0.f, 0.f};

  for (int r = 0; blockIdx.x + r * G < T; ++r) {
    int m0, n0;
    wv_origin(blockIdx.x + r * G, p.tiles_m, p.tiles_n, TM, TN, m0, n0);
    WaveLoader<!A_MN, TM> la;
    WaveLoader<B_KC, TN> lb;
    la.init(lda, lane);
    lb.init(ldb, lane);
    // Loads of this wave's step i into slot i % S.
    auto issue = [&](int i, uint8_t* slot) {
      const int kt = wave + WV_K * i;
      const bool ok = i < steps;
      la.issue(ra, lda, m0, kt, K, ok, slot);
      lb.issue(rb, ldb, n0, kt, K, ok, slot + ABYTES);
      if constexpr (MX) {
        const v4i xa = make_rsrc(p.mx_a, p.mx_a_bytes), xb = make_rsrc(p.mx_b, p.mx_b_bytes);
        const uint32_t oa = ((uint32_t)(kt * p.mx_groups_a + m0 / 64) * 64u + (uint32_t)lane) * 4u;
        const uint32_t ob = ((uint32_t)(kt * p.mx_groups_b + n0 / 64) * 64u + (uint32_t)lane) * 4u;
        load_lds4<0>(xa, ok ? oa : (uint32_t)xa.z, slot + ABYTES + BBYTES);
        load_lds4<0>(xb, ok ? ob : (uint32_t)xb.z, slot + ABYTES + BBYTES + 256);
      }
    };
    struct Frags {
      v8i a[MI], b[NI];
      int sa, sb;
    };
    auto read = [&](Frags& f, int i, uint8_t* slot) {
      if (wave + WV_K * i == KT_full && (krem & 15)) {  // the partial last step
        if constexpr (!A_MN) wv_zero_tail<TM>(slot, krem, lane);
        if constexpr (B_KC) wv_zero_tail<TN>(slot + ABYTES, krem, lane);
        wait_lgkmcnt<0>();
      }
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) f.a[mi] = wv_read_frag<!A_MN, TM, MX>(slot, 16 * mi, lane);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        f.b[ni] = wv_read_frag<B_KC, TN, MX>(slot + ABYTES, 16 * ni, lane);
      if constexpr (MX) {
        // byte i of a word: row block i of the tile (tiles start at 64-row groups)
        f.sa = *(const int*)(slot + ABYTES + BBYTES + 4 * lane);
        f.sb = *(const int*)(slot + ABYTES + BBYTES + 256 + 4 * lane);
      }
    };
    v4f acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Frags& f) {
      static_for<0, MI * NI>([&](auto I) {
        constexpr int mi = decltype(I)::value / NI, ni = decltype(I)::value % NI;
        acc[mi][ni] = mfma_s<FA, FB, MX, ni, mi>(f.b[ni], f.a[mi], acc[mi][ni], f.sb, f.sa);
      });
    };

    if (steps > 0) {
      static_for<0, S>([&](auto I) { issue(decltype(I)::value, mine + decltype(I)::value * SLOT); });
      Frags f[2];
      bool opens = first && r == 0 && header_begin(p, raw_scales);
      wait_vmcnt<(S - 1) * LPS>();
      read(f[0], 0, mine);
      wait_lgkmcnt<0>();
      __builtin_amdgcn_sched_barrier(0);
      issue(S, mine);
      int slot = 1;  // (i + 1) % S
      auto step = [&](const Frags& cur, Frags& next, int i) {
        uint8_t* s = mine + slot * SLOT;
        slot = slot + 1 == S ? 0 : slot + 1;
        wait_vmcnt<(S - 1) * LPS>();
        __builtin_amdgcn_sched_barrier(0);
        read(next, i + 1, s);
        multiply(cur);
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkmcnt<0>();  // the slot has been read
        __builtin_amdgcn_sched_barrier(0);
        issue(i + 1 + S, s);
      };
#pragma unroll 1
      for (int i = 0;;) {
        step(f[0], f[1], i);
        if (opens) {
          wait_vmcnt<2 * LPS>();  // (its words, before the loads of two steps)
          header_publish(p);
          opens = false;
        }
        if (++i >= steps) break;
        step(f[1], f[0], i);
        if (++i >= steps) break;
      }
      wait_vmcnt<0>();  // the zero loads past the last step
    } else {
      if (first && r == 0) header_open(p, raw_scales);
    }
    __syncthreads();

    // The partial tiles of the 4 waves, summed in wave order.
    float* part = (float*)ring;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        *(v4f*)(part + (wave * TM + 16 * mi + (lane & 15)) * RLD + 16 * ni + 4 * (lane >> 4)) =
            acc[mi][ni];
    __syncthreads();
    v4f v[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const float* q = part + (trow + 16 * j) * RLD + tcol;
      v4f s = *(const v4f*)q;
#pragma unroll
      for (int w = 1; w < WV_K; ++w) s += *(const v4f*)(q + w * TM * RLD);
      v[j] = s;
    }
    __syncthreads();  // (before the next tile's loads)

    const int m = m0 + trow, n = n0 + tcol;
    const int cols = min(N - n, 4);
    const bool inside = m0 + TM <= M && n0 + TN <= N;
    if (cols > 0) {
      if (fuse || p.acc_out || p.pre_out)
        ge_values(p, v, m, 16, n, cols, call_exponents(p, raw_scales), ge_bias(p, n));
      ge_fold(p, v, m, 16, cols, inside, lmax);
      if (p.epi == EPI_DIRECT)
        ge_store_codes(p, v, m, 16, n, cols, inside,
                       cast_rule(call_exponents(p, raw_scales).shift, p.sat != 0));
      else if (!p.single_pass)
        ge_store_inter(p, v, m, 16, n);
    }
    // (selects of values: a branch per tile would turn into a run-time index)
#pragma unroll
    for (int h = 0; h < kWaveHeld; ++h)
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) held[h][j][i] = r == h ? v[j][i] : held[h][j][i];
  }

  for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
  if (lane == 0) red[wave] = lmax;
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

  // Single pass: the held tiles are cast with the rescale of the whole
  // output's statistic. After an abort (the grid was not co-resident) every
  // workgroup writes its tiles to the intermediate and the last one casts.
  if (tid == 0) grid_wait(p, grid_arrive(p, wmax, G, ex.e_w), sp_word);
  __syncthreads();
  uint32_t amax_raw = sp_word[1];
  // Held tile h (a copy: one body for all of them) and where it lies.
  auto held_tile = [&](int h, v4f(&v)[NG], int& m, int& n, bool& inside)
      __attribute__((always_inline)) {
    int m0, n0;
    wv_origin(blockIdx.x + h * G, p.tiles_m, p.tiles_n, TM, TN, m0, n0);
    m = m0 + trow;
    n = n0 + tcol;
    inside = m0 + TM <= M && n0 + TN <= N;
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float x = held[0][j][i];
#pragma unroll
        for (int k = 1; k < kWaveHeld; ++k) x = h == k ? held[k][j][i] : x;
        v[j][i] = x;
      }
  };
  bool cast_all = false;
  if (sp_word[0] == SP_ABORTED) {
#pragma unroll 1
    for (int h = 0; blockIdx.x + h * G < T; ++h) {
      v4f v[NG];
      int m, n;
      bool inside;
      held_tile(h, v, m, n, inside);
      if (n < N) ge_store_inter(p, v, m, 16, n);
    }
    if (!last_writer(p, G, sp_word, amax_raw)) return;
    cast_all = true;
  }
  int e_out;
  const CastRule c = cast_rule(sp_shift(amax_raw, ex.e_w, p.e_cc, p.target, &e_out), p.sat != 0);
  if (tid == 0 && (blockIdx.x == 0 || cast_all)) {
    *p.out_scale = pow2_float(e_out);
    if (p.amax_out) *p.amax_out = __uint_as_float(amax_raw) * pow2_float(-p.e_cc);
  }
  if (cast_all) {
    ge_cast_all(p, tid, WV_THREADS, c);
    return;
  }
#pragma unroll 1
  for (int h = 0; blockIdx.x + h * G < T; ++h) {
    v4f v[NG];
    int m, n;
    bool inside;
    held_tile(h, v, m, n, inside);
    if (n < N) ge_store_codes(p, v, m, 16, n, min(N - n, 4), inside, c);
  }
}

template <bool A_MN, bool B_KC, bool MX>
struct WaveFamily {
  template <int FA, int FB>
  struct F {
    static hipError_t run(const GemmParams& p, hipStream_t s) {
      const dim3 g(p.grid), b(WV_THREADS);
      switch (wave_tile_rows(p.M)) {
        case 16: hipLaunchKernelGGL((wave_gemm_kernel<A_MN, B_KC, FA, FB, MX, 1>), g, b, 0, s, p); break;
        case 32: hipLaunchKernelGGL((wave_gemm_kernel<A_MN, B_KC, FA, FB, MX, 2>), g, b, 0, s, p); break;
        default: hipLaunchKernelGGL((wave_gemm_kernel<A_MN, B_KC, FA, FB, MX, 4>), g, b, 0, s, p); break;
      }
      return hipGetLastError();
    }
  };
};

}  // namespace scalify
