// Instantiations of the block-scaled FP8 GEMM for A stored [K][M] and B stored
// [K][N] (8-wave kernel).
#include "gemm8_kernel.h"

namespace scalify {

template <int FA, int FB>
struct Mx8 {
  static hipError_t run(const GemmParams& p, hipStream_t s) {
    const dim3 g(p.tiles_m * p.tiles_n), b(512);
    if (p.epi == EPI_DIRECT)
      hipLaunchKernelGGL((gemm8_kernel<true, false, FA, FB, EPI_DIRECT, false, true>), g, b, 0, s, p);
    else
      hipLaunchKernelGGL((gemm8_kernel<true, false, FA, FB, EPI_INTER32, false, true>), g, b, 0, s, p);
    return hipGetLastError();
  }
};

template <>
hipError_t launch_layout_mx<true, false>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<Mx8>(p, fa, fb, s);
}

}  // namespace scalify
