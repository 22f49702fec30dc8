// The backward products of fp32 layers by three bf16 pieces per value (linear_split.hip).
#pragma once

#include "linear_common.h"

namespace sar {

// dX [n, K] = dZ [n, F] W^T, F > 16; with op the rows of dZ are formed from the stored part (F whole pieces of 16 bytes,
// at most 16 heads).
int split_dx(const float* dZ, const RowsOp* op, const float* W, float* dX, int64_t n, int K, int F, hipStream_t st);

// Partial sums of dW = X^T dZ over at most most_slabs slabs of rows: partial [slabs, K, F].
int split_dw(const float* X, const float* dZ, const RowsOp* op, float* partial, int64_t n, int K, int F, int most_slabs,
             int* slabs, hipStream_t st);

}  // namespace sar
