// Instantiations of the small-output GEMM with MX block scales for A stored [K][M] and B stored [K][N].
#include "wave_gemm_kernel.h"

namespace scalify {

template <>
hipError_t launch_wave_layout<true, false, true>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<WaveFamily<true, false, true>::template F>(p, fa, fb, s);
}

}  // namespace scalify
