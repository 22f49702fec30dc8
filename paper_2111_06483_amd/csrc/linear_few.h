// The dense transform of few rows (linear_few.hip).
#pragma once

#include "linear_common.h"

namespace sar {

struct FewArgs {
    const void* A;     // [M, K], row stride K, contraction index contiguous
    int64_t M;
    const float* B;    // forward: W [K, N]; dX: W [N, K]
    void* C;           // [M, N], row stride N
    int K, N;
    // forward, fp32 rows of whole pieces: columns x . (W_h a1_h) and x . (W_h a2_h) beside the product
    const float* a1;   // [H, D] or null
    const float* a2;
    float* s1;         // [M, H] or null
    float* s2;
    int H, D;
};

// Whether a product of n rows is taken here: contraction of K values, N columns (and a tile of scores); wide: the column tiles
// that a wavefront of the other kernel would form.
bool few_rows(int dtype, int64_t n, int K, int N, bool scores, int wide);
// Z = X W (natural: the contraction in its natural order, as k_gemm_steps has it; otherwise k_gemm_skinny's).
int few_fwd(int dtype, const FewArgs& g, bool natural, hipStream_t st);

// dX and dW of one call together: dX = dZ W^T [n, K] (null: not wanted) and dW += X^T dZ (null: not wanted).  split: fp32
// dX by three bf16 pieces per value, as k_dx_split; otherwise by the fp32 instruction, as k_gemm_skinny or (natural) k_gemm_steps.
// work: [most_slabs, K, F] values.
struct FewBwd {
    const void* X;
    const void* dZ;
    const float* W;
    float* dW;
    void* dX;
    float* work;
    int64_t n;
    int K, F, most_slabs;
    bool split, natural;
};
// Whether the kernels of few rows take the call (formed: its rows are, by RowsOp).
bool few_rows_bwd(int dtype, const FewBwd& b, bool formed);
// slabs: partial sums of dW in work that are to be added up; 0: dW is complete.
int few_bwd(int dtype, const FewBwd& b, const RowsOp* op, int* slabs, hipStream_t st);

}  // namespace sar
