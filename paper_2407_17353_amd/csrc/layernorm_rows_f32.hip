// Single-read LayerNorm kernels for F32 inputs.
#include "layernorm_rows.h"

namespace scalify {

template <int OUTF, int WPR>
static void fwd(const LnParams& p, hipStream_t s) {
  const dim3 g(ln_rows_grid(p.R, WPR, 4)), b(LN_THREADS);
  if (p.D == 2048 * WPR) hipLaunchKernelGGL((ln_fwd_rows_kernel<kF32, OUTF, WPR, true>), g, b, 0, s, p);
  else hipLaunchKernelGGL((ln_fwd_rows_kernel<kF32, OUTF, WPR, false>), g, b, 0, s, p);
}

template <int OUTF>
static void fwd_out(const LnParams& p, hipStream_t s) {
  switch (ln_wpr(p.D)) {
    case 1: fwd<OUTF, 1>(p, s); break;
    case 2: fwd<OUTF, 2>(p, s); break;
    default: fwd<OUTF, 4>(p, s); break;
  }
}

template <>
void launch_ln_fwd_rows<kF32>(const LnParams& p, int out_dtype, hipStream_t s) {
  if (out_dtype == kE4M3) fwd_out<kE4M3>(p, s);
  else if (out_dtype == kE5M2) fwd_out<kE5M2>(p, s);
  else fwd_out<kF16>(p, s);
}

template <int DYF, int WPR>
static void bwd(const LnParams& p, hipStream_t s) {
  const dim3 g(ln_rows_grid(p.R, WPR, 3)), b(LN_THREADS);
  if (p.D == 2048 * WPR) hipLaunchKernelGGL((ln_bwd_rows_kernel<kF32, DYF, WPR, true>), g, b, 0, s, p);
  else hipLaunchKernelGGL((ln_bwd_rows_kernel<kF32, DYF, WPR, false>), g, b, 0, s, p);
}

template <int DYF>
static void bwd_dy(const LnParams& p, hipStream_t s) {
  switch (ln_wpr(p.D)) {
    case 1: bwd<DYF, 1>(p, s); break;
    case 2: bwd<DYF, 2>(p, s); break;
    default: bwd<DYF, 4>(p, s); break;
  }
}

template <>
void launch_ln_bwd_rows<kF32>(const LnParams& p, hipStream_t s) {
  if (p.dy_fmt == kF16) bwd_dy<kF16>(p, s);
  else if (p.dy_fmt == kF32) bwd_dy<kF32>(p, s);
  else if (p.dy_fmt == kE4M3) bwd_dy<kE4M3>(p, s);
  else bwd_dy<kE5M2>(p, s);
}

}  // namespace scalify
