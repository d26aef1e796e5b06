// Dispatch of the small-output GEMM over the storage orders of A and B.
#include "wave_gemm.h"

namespace scalify {

hipError_t launch_wave_gemm(const GemmParams& p, bool a_mn, bool b_kc, int fa, int fb,
                            hipStream_t s) {
  if (p.mx_a) {
    if (!a_mn && b_kc) return launch_wave_layout<false, true, true>(p, fa, fb, s);
    if (!a_mn && !b_kc) return launch_wave_layout<false, false, true>(p, fa, fb, s);
    if (a_mn && b_kc) return launch_wave_layout<true, true, true>(p, fa, fb, s);
    return launch_wave_layout<true, false, true>(p, fa, fb, s);
  }
  if (!a_mn && b_kc) return launch_wave_layout<false, true, false>(p, fa, fb, s);
  if (!a_mn && !b_kc) return launch_wave_layout<false, false, false>(p, fa, fb, s);
  if (a_mn && b_kc) return launch_wave_layout<true, true, false>(p, fa, fb, s);
  return launch_wave_layout<true, false, false>(p, fa, fb, s);
}

}  // namespace scalify
