// Host side of the 128-row-tile GEMM (mid_gemm_kernel.h).
#pragma once
#include "gemm_choice.h"
#include "kernels.h"

namespace scalify {

// Launch on p (tiles_m, tiles_n, grid and epi set for the tile).
hipError_t launch_mid_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb, MidTile tile,
                           hipStream_t s);
template <bool A_MN, bool B_KC>
hipError_t launch_mid_layout(const GemmParams& p, int fa, int fb, MidTile tile, hipStream_t s);

}  // namespace scalify
