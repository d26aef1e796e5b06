// Host side of the small-output GEMM (wave_gemm_kernel.h): its launch.
#pragma once
#include "gemm_choice.h"
#include "kernels.h"

namespace scalify {

// Launch on p (tiles_m, tiles_n, grid and epi set for this kernel).
hipError_t launch_wave_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb,
                            hipStream_t s);
template <bool A_MN, bool B_KC, bool MX>
hipError_t launch_wave_layout(const GemmParams& p, int fa, int fb, hipStream_t s);

}  // namespace scalify
