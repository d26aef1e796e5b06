// Instantiations of the 128-row-tile GEMM for A stored [K][M] and B stored [K][N].
#include "mid_gemm_kernel.h"

namespace scalify {

template <>
hipError_t launch_mid_layout<true, false>(const GemmParams& p, int fa, int fb, MidTile tile, hipStream_t s) {
  if (tile == MID_256) return by_formats<MidFamily<true, false, 8, 3>::template F>(p, fa, fb, s);
  if (tile == MID_128) return by_formats<MidFamily<true, false, 4, 4>::template F>(p, fa, fb, s);
  return by_formats<MidFamily<true, false, 4, 2>::template F>(p, fa, fb, s);
}

}  // namespace scalify
