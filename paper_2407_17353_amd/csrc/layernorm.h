// Internal interface of the scaled LayerNorm kernels (layernorm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scalify {

// Rows of D <= 8192 values, row-major.
struct LnParams {
  const void* x;        // [R][ldx], format x_fmt
  int64_t ldx;
  int x_fmt;
  const void* dy;       // backward: [R][lddy], format dy_fmt
  int64_t lddy;
  int dy_fmt;
  const float* gamma;   // [D] or NULL (1)
  const float* beta;    // [D] or NULL (0)
  void* out;            // forward y / backward dx codes [R][ldo]
  int64_t ldo;
  float* pre_out;       // optional fp32 [R][D]: the values before the cast
  int64_t R;
  int D;
  float eps;
  int sat, target, mode;  // backward rescale: mode 1 = amax, 0 = none
  uint32_t* hdr;        // backward: workspace header
  uint64_t tag;         // backward: the call's tag in it (stat_header.h)
  const float* s_dy;    // backward: scales of dy and x (NULL = 1)
  const float* s_x;
  float* partial;       // backward: per-row numbers [R][4], then [row tiles][2][stride]
  float* out_scale;
  float* amax_out;      // backward: optional amax of |dx|
  float* dgamma;        // backward: optional [D]
  float* dbeta;         // backward: optional [D]
};

constexpr int kLayerNormMaxD = 8192;

// Row stride of the backward's partial parameter gradients (16-float aligned).
__host__ __device__ inline int64_t layernorm_param_stride(int64_t D) { return (D + 15) / 16 * 16; }
// Backward workspace after the header, in floats: per-row numbers (4 R) and
// per-row-tile partial parameter gradients.
int64_t layernorm_ws_floats(int64_t R, int64_t D);
hipError_t launch_layernorm_fwd(const LnParams& p, int out_dtype, hipStream_t s);
hipError_t launch_layernorm_bwd(const LnParams& p, int out_dtype, hipStream_t s);

// Families, each input format in a source file of its own:
//   launch_ln_fwd_rows, launch_ln_bwd_rows: rows read once (layernorm_rows.h);
//   launch_ln_apply: the backward's cast of dx and partial parameter sums.
template <int XF>
void launch_ln_fwd_rows(const LnParams& p, int out_dtype, hipStream_t s);
template <int XF>
void launch_ln_bwd_rows(const LnParams& p, hipStream_t s);
template <int XF>
void launch_ln_apply(const LnParams& p, int out_dtype, hipStream_t s);
// Waves per row of the row kernels, and their workgroups for `wpr`.
inline int ln_wpr(int D) { return D <= 2048 ? 1 : (D <= 4096 ? 2 : 4); }
int ln_rows_grid(int64_t R, int wpr, int per_cu);
int64_t layernorm_row_tiles(int64_t R);

}  // namespace scalify
