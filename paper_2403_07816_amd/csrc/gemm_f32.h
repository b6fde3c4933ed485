// Entry points of the fp32 grouped-GEMM path (see gemm_f32.hip).
#pragma once
#include "common.h"

namespace btx {
// the number of rows that the interface documents for fp32 (R/64 + E <= 65535); the kernels' grids would take more
bool f32_rows_ok(int R, int E);
// partial sums of dg per grouped row that f32_bwd_act leaves (one per column tile)
int f32_bwd_act_partials(int f);
// xs / dys: token rows, read through perm.  row_bytes: [R], scratch that f32_bwd_act fills for the weight gradients (NULL: none wanted)
int f32_up_swiglu(const RowSource& xs, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh, void* h1,
                  void* h3, void* act, hipStream_t s);
// sums: scratch for the sums of K slices, of f32_down_sums_bytes() (f32_bwd_dx_sums_bytes() in the backward pass); NULL when that is 0
size_t f32_down_sums_bytes(const FfShapes& sh);
size_t f32_bwd_dx_sums_bytes(const FfShapes& sh);
// slices: see launch_down()
int f32_down(const void* act, const void* W2, const int32_t* off, const FfShapes& sh, void* y, void* sums, int* slices,
             hipStream_t s);
// Both products of a small layer in one launch: y is left as the sums of slices of f, [slice][R, d], f32_ff_slices() of them (0: not
// such a layer, or more than `most`)
int f32_ff_slices(const FfShapes& sh, int64_t most);
int f32_ff(const RowSource& xs, const void* W1, const void* W3, const void* W2, const int32_t* off, const FfShapes& sh, void* h1, void* h3,
           void* sums, hipStream_t s);
int f32_bwd_act(const RowSource& dys, const void* W2, const void* h1, const void* h3, const float* gates,
                const int32_t* perm, const int32_t* off, const FfShapes& sh, void* dh1, void* dh3, void* ga,
                uint32_t* row_bytes, float* dg_part, hipStream_t s);
int f32_bwd_dx(const void* dh1, const void* dh3, const void* W1, const void* W3, const int32_t* off, const FfShapes& sh,
               void* dxs, void* sums, hipStream_t s);
// the same with the weight gradients
int f32_bwd_dx_dw(const RowSource& xs, const RowSource& dys, const void* dh1, const void* dh3, const void* ga, const void* W1,
                  const void* W3, const int32_t* off, const FfShapes& sh, uint32_t* row_bytes, void* dxs, void* sums, void* dW1,
                  void* dW3, void* dW2, const RouterDs* ds, hipStream_t s);
}  // namespace btx
