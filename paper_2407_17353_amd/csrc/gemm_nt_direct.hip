// Instantiations of the scaled FP8 GEMM with the direct cast (output scale known before the
// GEMM: delayed or no rescale) for
// A stored [M][K] and B stored [N][K].
#include "gemm4_kernel.h"

namespace scalify {

template <>
hipError_t launch_layout_direct<false, true>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<DirectFamily<false, true, false>::template F>(p, fa, fb, s);
}

}  // namespace scalify
