// The LayerNorm backward's apply kernel for F16 inputs.
#include "layernorm_apply.h"

namespace scalify {

template <int DYF>
static void apply(const LnParams& p, int out_dtype, dim3 g, dim3 b, hipStream_t s) {
  if (out_dtype == kE4M3) hipLaunchKernelGGL((ln_bwd_apply_kernel<kF16, DYF, kE4M3>), g, b, 0, s, p);
  else if (out_dtype == kE5M2) hipLaunchKernelGGL((ln_bwd_apply_kernel<kF16, DYF, kE5M2>), g, b, 0, s, p);
  else hipLaunchKernelGGL((ln_bwd_apply_kernel<kF16, DYF, kF16>), g, b, 0, s, p);
}

template <>
void launch_ln_apply<kF16>(const LnParams& p, int out_dtype, hipStream_t s) {
  // It also writes the output scale: at least one workgroup.
  const int cols = (p.D + LN_TILE_COLS - 1) / LN_TILE_COLS;
  const dim3 g(cols < 1 ? 1 : cols, (unsigned)layernorm_row_tiles(p.R)), b(LN_TILE_THREADS);
  if (p.dy_fmt == kF16) apply<kF16>(p, out_dtype, g, b, s);
  else if (p.dy_fmt == kF32) apply<kF32>(p, out_dtype, g, b, s);
  else if (p.dy_fmt == kE4M3) apply<kE4M3>(p, out_dtype, g, b, s);
  else apply<kE5M2>(p, out_dtype, g, b, s);
}

}  // namespace scalify
