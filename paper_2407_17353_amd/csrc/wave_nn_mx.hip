// Instantiations of the small-output GEMM with MX block scales for A stored [M][K] and B stored [K][N].
#include "wave_gemm_kernel.h"

namespace scalify {

template <>
hipError_t launch_wave_layout<false, false, true>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<WaveFamily<false, false, true>::template F>(p, fa, fb, s);
}

}  // namespace scalify
