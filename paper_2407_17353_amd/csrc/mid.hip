// Dispatch of the 128-row-tile GEMM over the storage orders of A and B.
#include "mid_gemm.h"

namespace scalify {

hipError_t launch_mid_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb, MidTile tile,
                           hipStream_t s) {
  if (!a_mn && b_kc) return launch_mid_layout<false, true>(p, fa, fb, tile, s);
  if (!a_mn && !b_kc) return launch_mid_layout<false, false>(p, fa, fb, tile, s);
  if (a_mn && b_kc) return launch_mid_layout<true, true>(p, fa, fb, tile, s);
  return launch_mid_layout<true, false>(p, fa, fb, tile, s);
}

}  // namespace scalify
