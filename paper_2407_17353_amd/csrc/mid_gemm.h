// Host side of the 128-row-tile GEMM (mid_gemm_kernel.h).
#pragma once
#include "kernels.h"

namespace scalify {

constexpr int kMidTM = 128;  // output rows of a tile

// Tiles and pipelines: 128 x 256 (3 stages), 128 x 128 (4 stages), one
// workgroup per CU; 128 x 128 with 2 stages, two workgroups per CU, whose
// epilogues and main loops overlap.
enum MidTile { MID_256, MID_128, MID_128_PAIR };

// Launch on p (tiles_m, tiles_n, grid and epi set for the tile).
hipError_t launch_mid_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb, MidTile tile,
                           hipStream_t s);
template <bool A_MN, bool B_KC>
hipError_t launch_mid_layout(const GemmParams& p, int fa, int fb, MidTile tile, hipStream_t s);

}  // namespace scalify
