// Instantiations of the scaled FP8 GEMM with the fused residual add, activation and channel
// scales (8-wave kernel) for
// A stored [M][K] and B stored [K][N].
#include "gemm8_kernel.h"

namespace scalify {

template <>
hipError_t launch_layout_fused<false, false>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<FusedFamily<false, false>::template F>(p, fa, fb, s);
}

}  // namespace scalify
