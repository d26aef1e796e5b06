// Instantiations of the scaled FP8 GEMM with the pre-cast intermediate (GEMM + cast kernel) for
// A stored [K][M] and B stored [N][K].
#include "gemm4_kernel.h"

namespace scalify {

template <>
hipError_t launch_layout<true, true>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<PlainFamily<true, true>::template F>(p, fa, fb, s);
}

}  // namespace scalify
