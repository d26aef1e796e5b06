// Host side of the small-output GEMM (wave_gemm_kernel.h): which calls take
// it, and its launch.
#pragma once
#include "kernels.h"

namespace scalify {

constexpr int kWaveTN = 64;   // output columns of a tile
constexpr int kWaveHeld = 4;  // tiles a workgroup can hold through the single pass

// Rows of a tile: the smallest of 16, 32, 64 that holds M, else 64.
inline int wave_tile_rows(int64_t M) { return M <= 16 ? 16 : (M <= 32 ? 32 : 64); }

// Launch on p (tiles_m, tiles_n, grid and epi set for this kernel).
hipError_t launch_wave_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb,
                            hipStream_t s);
template <bool A_MN, bool B_KC, bool MX>
hipError_t launch_wave_layout(const GemmParams& p, int fa, int fb, hipStream_t s);

}  // namespace scalify
