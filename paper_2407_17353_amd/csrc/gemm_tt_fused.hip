// Instantiations of the scaled FP8 GEMM with the fused residual add, activation and channel
// scales (8-wave kernel) for
// A stored [K][M] and B stored [N][K].
#include "gemm8_kernel.h"

namespace scalify {

template <>
hipError_t launch_layout_fused<true, true>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<FusedFamily<true, true>::template F>(p, fa, fb, s);
}

}  // namespace scalify
