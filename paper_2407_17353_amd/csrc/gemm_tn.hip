// Instantiations of the scaled FP8 GEMM with the pre-cast intermediate (GEMM + cast kernel) for
// A stored [K][M] and B stored [K][N].
#include "gemm4_kernel.h"

namespace scalify {

template <>
hipError_t launch_layout<true, false>(const GemmParams& p, int fa, int fb, hipStream_t s) {
  return by_formats<PlainFamily<true, false>::template F>(p, fa, fb, s);
}

}  // namespace scalify
