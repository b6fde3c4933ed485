// Entry points of the bf16 MFMA grouped-GEMM path (see gemm_mfma.hip).
#pragma once
#include "common.h"

namespace btx {
// raises the dynamic-LDS limit of every kernel instantiation on the current device (not capturable)
int mfma_prepare();
// the weight-gradient products address 255 rows of the transposed, padded operands with 32-bit byte offsets
bool mfma_rows_ok(int R, int E);
// and the k rows of a k tile of the operands in row order likewise (direct: mfma_dw_direct())
bool mfma_dw_ok(int R, int f, bool direct);
int mfma_bwd_act_partials(const FfShapes& sh);
int mfma_bwd_act_partials_most(int f);
// gathered A rows need every byte offset inside the source to fit 32 bits
bool mfma_gather_ok(int T, int d);
// partial: scratch for the sums of K slices, of mfma_forward_split_bytes() (mfma_backward_split_bytes() in mfma_bwd_dx); NULL
// when that is 0
size_t mfma_forward_split_bytes(const FfShapes& sh);
size_t mfma_backward_split_bytes(const FfShapes& sh);
int mfma_up_swiglu(const RowSource& xs, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh,
                   void* h1, void* h3, void* act, void* partial, hipStream_t s);
// slices: see launch_down()
int mfma_down(const void* act, const void* W2, const int32_t* off, const FfShapes& sh, void* y, void* partial,
              int* slices, hipStream_t s);
// dh1, dh3: [R,f], rows mfma_act_pitch() apart; ga: like them, or with ga_transposed [f][mfma_dw_pitch(R, E)], experts' rows padded with zeros to
// multiples of 64 (for dW2; NULL when no weight gradients are wanted)
int mfma_bwd_act(const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                 const int32_t* perm, const int32_t* off, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                 bool ga_transposed, uint32_t* row_bytes, float* dg_part, hipStream_t s);
int mfma_bwd_dx(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off,
                const FfShapes& sh, void* dxs, void* partial, hipStream_t s);
// Weight gradients.  mfma_dw_direct(): of few rows per expert, from token rows (found by row_bytes) and ga in row order; else
// xs, dys without perm: [d][mfma_dw_pitch(R, E)], laid out like the transposed ga above
bool mfma_dw_direct(const FfShapes& sh, int dW_dtype);
int mfma_dw_pitch(int R, int E);
// elements from a row of act, dh1, dh3 or ga (in row order) to the next
int mfma_act_pitch(int f);
int mfma_bwd_dw13(int dW_dtype, const RowSource& xs, const void* dh1, const void* dh3, const int32_t* off, const FfShapes& sh, void* dW1,
                  void* dW3, hipStream_t s);
// row_bytes: dys are token rows, found by it (mfma_dw2_rows(); NULL: transposed like xs)
bool mfma_dw2_rows(const FfShapes& sh);
int mfma_bwd_dw2(int dW_dtype, const void* ga, const RowSource& dys, const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dW2,
                 hipStream_t s);
int mfma_bwd_dw_direct(int dW_dtype, const RowSource& xs, const RowSource& dys, const void* dh1, const void* dh3, const void* ga,
                       const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dW1, void* dW3, void* dW2,
                       const RouterDs* ds, hipStream_t s);
}  // namespace btx
