// Which GEMM kernel takes a matmul, and its output tile: host code alone.
#pragma once
#include <stdint.h>

namespace scalify {

// wave_gemm_kernel.h: 16, 32 or 64 x 64 tiles.
constexpr int kWaveTN = 64;   // output columns of a tile
constexpr int kWaveHeld = 2;  // tiles a workgroup can hold through the single pass
// Rows of a tile: the smallest of 16, 32, 64 that holds M, else 64.
inline int wave_tile_rows(int64_t M) { return M <= 16 ? 16 : (M <= 32 ? 32 : 64); }

// mid_gemm_kernel.h. Tiles and pipelines: 128 x 256 (3 stages), 128 x 128 (4
// stages), one workgroup per CU; 128 x 128 with 2 stages, two workgroups per
// CU, whose epilogues and main loops overlap.
constexpr int kMidTM = 128;  // output rows of a tile
enum MidTile { MID_256, MID_128, MID_128_PAIR };

// The GEMM kernel of a call and its output tile: gemm4_kernel.h (GEMM_BIG;
// gemm8_kernel.h for block scales of A [K][M] with B [K][N]), gemm8_kernel.h
// (GEMM_FUSED), mid_gemm_kernel.h, wave_gemm_kernel.h.
enum GemmKind { GEMM_BIG, GEMM_FUSED, GEMM_MID, GEMM_WAVE };
struct GemmChoice {
  GemmKind kind;
  int tm, tn;
  int64_t tiles;
  MidTile mid;
  int resident;  // workgroups that a CU holds
};

// The rule, on the counts of tiles that each kernel would have (times in us,
// AMAX, [M][K] x [K][N], 256 CUs, the two kernels in the order named):
// - Up to one 16/32/64 x 64 tile per CU: the wave kernel, whose 4 waves split
//   K. 64x4096x4096 (64 tiles) against 128 x 128 tiles 16.1 / 25.4,
//   256x4096x4096 (256) 22.2 / 24.5, 256x4096x8192 without rescale 25 / 47;
//   with one more tile per CU it loses, 512x4096x1024 (512) 23.2 / 15.7.
//   Block scales, which the 128-row kernel does not have, take it up to two
//   tiles per CU, against 256 x 256 tiles: 512x4096x4096 34.5 / 53.6, but
//   1024x4096x1024 (1024) 35.3 / 25.0. Not the last of them while K is too short
//   for the split: 2048x1024xK (512), K 64 20.9 / 17.9, 256 21.2 / 17.9 (without
//   rescale 15.9 / 15.8), 512 22.6 / 20.3 (15.8 / 17.4); 384x4096x256 (384) 17.8
//   / 19.5.
// - Up to one 128 x 256 tile per CU: the 128-row kernel, a 256 x 256 grid
//   leaving half the chip idle. 128 x 128 tiles, two workgroups to a CU, while
//   K is short: 1024x4096x1024 19.4 against 20.9 of 128 x 256 and 23.4 of
//   256 x 256 tiles. A deeper ring (one workgroup to a CU) or the larger tile
//   for long K: 2048x2048x8192 56.6 / 51.9, 2048x4096x8192 72.3 / 63.7
//   (256 x 256: 87.4).
//   With a statistic, the two atomics of each workgroup on one line weigh where
//   there are many and K is short: 256 x 256 tiles again. AMAX, against these,
//   512 workgroups, 2048x4096xK: K 64 22.9 / 19.8, 512 25.2 / 22.3, 1024 27.2 /
//   26.2, 1536 30.1 / 31.0; 384 workgroups, 1536x4096xK: K 64 19.5 / 18.7, 512
//   21.5 / 21.1, 768 22.1 / 23.3.
// - Else 256 x 256 tiles; with a fused epilogue, which that kernel has only in
//   its slower 8-wave form, 128 x 128 tiles where these fill their rounds of
//   512 that much better than 256 x 256 tiles fill rounds of 256 (a round of
//   them takes 9/16 of the other's time): bias and GELU 3001x8192x2048 (3 and
//   2 rounds) 93.7 against 100.7, 4096x8192x2048 (4 and 2) 118 / 112,
//   8192x8192x2048 304 / 243. (Without one: 3001x8192x2048 71.7 / 65.4.) Not
//   where operands and fp32 intermediate outgrow the 256 MiB last-level cache,
//   from which the smaller tiles read their panels more often: AMAX
//   3001x12288x5504 (231 MB) 247 / 255, 2048x12288x11008 (258 MB) 329 / 286,
//   3001x12288x8192 (272 MB) 355 / 336; direct casts, without an intermediate,
//   304 / 331 at the last one.
// Calls of one size and kind sum K in one order in every mode: all kernels but
// the wave kernel and the block-scaled ones go through K alike. Calls of other
// sizes need not: the wave kernel sums four interleaved shares of K.
// amax: dynamic rescale; statistic: it or another call that reports one.
inline GemmChoice gemm_choice(int64_t M, int64_t N, int64_t K, int cus, bool fused, bool mx, bool amax,
                              bool statistic) {
  auto make = [&](GemmKind k, int tm, int tn, MidTile t = MID_256) {
    return GemmChoice{k, tm, tn, ((M + tm - 1) / tm) * ((N + tn - 1) / tn), t, t == MID_128_PAIR ? 2 : 1};
  };
  const GemmChoice big = make(fused ? GEMM_FUSED : GEMM_BIG, 256, 256);
  const GemmChoice wave = make(GEMM_WAVE, wave_tile_rows(M), kWaveTN);
  const GemmChoice mid8 = make(GEMM_MID, kMidTM, 256, MID_256);
  const GemmChoice mid4 = make(GEMM_MID, kMidTM, 128, MID_128);
  const GemmChoice pair = make(GEMM_MID, kMidTM, 128, MID_128_PAIR);
  if (mx && K <= 256 && 4 * wave.tiles > 7 * cus) return big;
  if (mx) return wave.tiles <= kWaveHeld * cus ? wave : big;
  if (wave.tiles <= cus) return wave;
  if (mid8.tiles <= cus && !fused && statistic &&
      ((K <= 512 && 2 * pair.tiles >= 3 * cus) || (K <= 1024 && 4 * pair.tiles > 7 * cus)))
    return big;
  if (mid8.tiles <= cus) return K < 4096 ? pair : mid4.tiles <= cus ? mid4 : mid8;
  if (!fused) return big;
  if (amax && M * K + K * N + 4 * M * N > 240000000) return big;
  const int64_t big_rounds = (big.tiles + cus - 1) / cus, pair_rounds = (pair.tiles + 2 * cus - 1) / (2 * cus);
  return 9 * pair_rounds < 16 * big_rounds ? pair : big;
}

}  // namespace scalify
