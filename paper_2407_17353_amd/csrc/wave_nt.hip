// Instantiations of the small-output GEMM for A stored [M][K] and B stored [N][K].
#include "wave_gemm_kernel.h"

namespace scalify {

template <>
hipError_t launch_wave_layout<false, true, false>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<WaveFamily<false, true, false>::template F>(p, fa, fb, s);
}

}  // namespace scalify
