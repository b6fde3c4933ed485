// Dispatch of the expert-FFN stages to the kernels that implement them, by storage type:
// gemm_f32.hip for fp32, gemm_mfma.hip for bf16.
#include "common.h"
#include "gemm_f32.h"
#include "gemm_mfma.h"

namespace btx {

int ff_prepare() { return mfma_prepare(); }

// bf16 with a d or f that is not a multiple of 32 keeps the documented limit of the fp32 path
bool ff_rows_supported(int dtype, int R, int d, int f, int E) {
  if (dtype != BTX_BF16) return f32_rows_ok(R, E);
  return mfma_rows_ok(R, E) && ((d % 32 == 0 && f % 32 == 0 && d >= 64 && f >= 64) || f32_rows_ok(R, E));
}

bool ff_dw_supported(int dtype, const FfShapes& sh, bool direct) { return dtype != BTX_BF16 || mfma_dw_ok(sh.R, sh.f, direct); }

bool ff_dw_transposed(int dtype) { return dtype == BTX_BF16; }
bool ff_dw_direct(int dtype, int dW_dtype, const FfShapes& sh, bool gather_fused) {
  return dtype != BTX_BF16 || (gather_fused && mfma_dw_direct(sh, dW_dtype));
}
bool ff_dw2_rows(int dtype, int T, const FfShapes& sh) { return dtype == BTX_BF16 && ff_gather_fused(dtype, T, sh.d) && mfma_dw2_rows(sh); }
int ff_dw_pitch(int R, int E) { return mfma_dw_pitch(R, E); }
int ff_act_pitch(int dtype, int f) { return dtype == BTX_BF16 ? mfma_act_pitch(f) : f; }

bool ff_gather_fused(int dtype, int T, int d) { return dtype != BTX_BF16 || mfma_gather_ok(T, d); }

int bwd_act_partials(int dtype, const FfShapes& sh) {
  return dtype == BTX_BF16 ? mfma_bwd_act_partials(sh) : f32_bwd_act_partials(sh.f);
}

int bwd_act_partials_most(int dtype, int f) { return dtype == BTX_BF16 ? mfma_bwd_act_partials_most(f) : f32_bwd_act_partials(f); }

size_t ff_forward_split_bytes(int dtype, const FfShapes& sh) {
  return dtype == BTX_BF16 ? mfma_forward_split_bytes(sh) : f32_down_sums_bytes(sh);
}
size_t ff_backward_split_bytes(int dtype, const FfShapes& sh) {
  return dtype == BTX_BF16 ? mfma_backward_split_bytes(sh) : f32_bwd_dx_sums_bytes(sh);
}

int launch_up_swiglu(int dtype, const RowSource& xs, const void* W1, const void* W3, const int32_t* offsets,
                     const FfShapes& sh, void* h1, void* h3, void* act, void* partial, hipStream_t s) {
  if (dtype == BTX_BF16) return mfma_up_swiglu(xs, W1, W3, offsets, sh, h1, h3, act, partial, s);
  return f32_up_swiglu(xs, W1, W3, offsets, sh, h1, h3, act, s);
}
int launch_down(int dtype, const void* act, const void* W2, const int32_t* offsets, const FfShapes& sh, void* y,
                void* partial, int* slices, hipStream_t s) {
  if (dtype == BTX_BF16) return mfma_down(act, W2, offsets, sh, y, partial, slices, s);
  return f32_down(act, W2, offsets, sh, y, partial, slices, s);
}
int launch_bwd_act(int dtype, const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                   const int32_t* perm, const int32_t* offsets, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                   bool want_dw, bool ga_transposed, uint32_t* row_bytes, float* dg_part, hipStream_t s) {
  if (!want_dw) ga = nullptr;
  if (dtype == BTX_BF16) return mfma_bwd_act(dys, W2, h1, h3, gates, perm, offsets, sh, dh1, dh3, ga, ga_transposed, row_bytes, dg_part, s);
  return f32_bwd_act(dys, W2, h1, h3, gates, perm, offsets, sh, dh1, dh3, ga, row_bytes, dg_part, s);
}
int launch_bwd_dx(int dtype, const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* offsets,
                  const FfShapes& sh, void* dxs, void* partial, hipStream_t s) {
  if (dtype == BTX_BF16) return mfma_bwd_dx(dh1, dh3, W1, W3, offsets, sh, dxs, partial, s);
  return f32_bwd_dx(dh1, dh3, W1, W3, offsets, sh, dxs, partial, s);
}

}  // namespace btx
