// The fp32 products of the dense transform on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values, x = x1 + x2 + x3 (24 significant bits in pieces of 8, each
// rounded to nearest), and the product of two pieces is exact in fp32.  Of the nine
// partial products x3 y2, x2 y3 and x3 y3 are left out (below 2^-23 of |x y|, of either sign); the other six are added
// smallest first:
//     x3 y1, x1 y3, x2 y2, x2 y1, x1 y2, x1 y1.
// V_MFMA_F32_32X32X16_BF16 takes 16 contraction values where V_MFMA_F32_32X32X2_F32 takes 2, in half the cycles, so
// six of them do in 192 cycles what the fp32 instruction does in 512.  Errors stand at the kernels.
//
// Infinities, NaN and finite values beyond bf16's largest (3.39e38) have no such sum: their pieces hold a NaN, so
// every result they take part in is NaN.  Nor has a value below 2^-110, whose last bits are smaller than bf16's smallest
// value.  And pieces rounded up may carry a result that ends below fp32's largest value beyond it on the way.  Where results
// hold a NaN or an infinity or operands such a small value (zero is none), a wavefront (k_dx_split) or a workgroup
// (k_dw_split) forms its results again with the fp32 instruction from the operands themselves: slower, with fp32's own
// results.
#include <algorithm>

#include "linear_pieces.h"
#include "linear_split.h"
#include "sar_internal.h"

namespace {

using namespace sar;

// ---- dX = dZ W^T ---------------------------------------------------------------
//
// A wavefront keeps 32 rows of the result, NT tiles of 32 columns wide, in registers.  Its rows of A come straight
// from memory in steps of 16 contraction values (32 bytes per lane: row l%32, values 8 (l/32) ..), two steps ahead, and
// are split in registers.  The small operand passes through LDS in the same steps, in the order the fragments are
// consumed: the next step's values, loaded during this one, are split once per workgroup of four wavefronts and written
// to the other buffer after this step's products, so there is one barrier per step.  A workgroup takes row block after
// row block, and the first steps of the next block travel while this one is stored.  Two to four workgroups per CU,
// which do not wait for each other; the slabs of the same rows run on one XCD, whose L2 serves the rows again.
//
// The matrix cores cut a product's bits below the sum's instead of rounding them, always downwards.  Small terms added to a
// long sum left errors of one sign: their mean was 0.06 to 0.14 of their standard deviation (normal values, 17 to 512
// products a result; the fp32 instruction: 0.001), and up to 0.44 of it in a column of non-negative values, and the next
// layer sums dX over all nodes.  So a step's 16 products are summed by themselves, small terms first, and added by vector
// instructions, which round to nearest; and every other row and step takes A with the other sign.  Error against 64-bit
// sums, fp32 instruction / here: 17 products 7.7e-8 / 4.2e-8, 64 1.5e-7 / 5.2e-8, 256 2.9e-7 / 8.4e-8, 400 3.6e-7 / 1.0e-7;
// uniform in (0, 1) 6.5e-8 / 4.1e-8, 1.2e-7 / 4.1e-8, 2.2e-7 / 6.0e-8, 2.9e-7 / 7.6e-8.
//
// FUSE: the rows of A are formed where they are split (RowsOp).
//
// Bound by what a SIMD can issue: of its cycles at 306250 rows 256 -> 256, 1.8 GHz under this load, the matrix instructions
// take 47% and the vector instructions (splitting, adding, checking) 46%, and they overlap little; by memory latency in
// narrow products.  dX against the fp32 instruction, plain / with formed rows, us: 306250 rows 256 -> 256
// 351 / 362 -> 291 / 306, 256 -> 100 181 / 196 -> 145 / 163; 2450000 rows 400 -> 400 7950 -> 5700; 75000 rows 128 -> 128
// 40 / 42 -> 26 / 32; 8000 rows 256 -> 256 33 / 37 -> 17 / 21; 100 rows 128 -> 100 17 / 19 -> 10 / 12.  (Also measured: one workgroup of eight wavefronts per CU, of which four split before they
// multiply and four after, the same within 5%, small products slower; steps of 32 values and results stored during the
// next block's steps, 10 to 20% slower.)
constexpr int kThreads = 256;
constexpr int kBlockRows = 128;
constexpr int kStep = 16;
constexpr int kFewWorkgroups = 192;
constexpr int kMaxRowsHeads = 16;    // heads of a formed row (a wavefront's 32 x H values of ds: 8 registers)

struct SplitArgs {
    const float* A;    // [M, K], row stride lda, contraction index contiguous
    int64_t lda, M;
    const float* B;    // [N, K], contraction index contiguous
    float* C;          // [M, N], row stride ldc
    int64_t ldc;
    int K, N, steps, slabs;
    RowsOp op;
};

// Workgroups per CU (wavefronts per SIMD) that the registers allow.
constexpr int dx_waves(int nt, bool fuse) { return fuse ? (nt <= 2 ? 3 : 2) : nt <= 2 ? 4 : nt <= 4 ? 3 : 2; }

template <int NT, bool FUSE>
__global__ __launch_bounds__(kThreads, dx_waves(NT, FUSE)) void k_dx_split(SplitArgs g)
{
    constexpr int kBuf = NT * 3 * 64;                               // units of a step
    constexpr int kPer = (NT * 64 + kThreads - 1) / kThreads;       // items of 8 values of one column per thread
    extern __shared__ __attribute__((aligned(16))) uint4 split_lds[];
    uint4* frag = split_lds;                                        // [2][kBuf]
    float* extra = reinterpret_cast<float*>(split_lds + 2 * kBuf);  // FUSE: a_r and the wavefronts' ds
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, gq = lane >> 5;
    const int64_t row_blocks = (g.M + kBlockRows - 1) / kBlockRows;
    // blocks 8 apart share an XCD: the slabs of one row block, whose rows the XCD's L2 serves the second time
    const int64_t stride = gridDim.x / g.slabs;
    int64_t rb = (int64_t)(blockIdx.x / (8 * g.slabs)) * 8 + blockIdx.x % 8;
    const int slab = (int)(blockIdx.x / 8 % g.slabs), n0 = slab * NT * 32;
    if (rb >= row_blocks) return;

    const int k_last = g.K - 4, rest = g.K % 4;
    auto row_index = [&](int64_t b) SAR_INLINE { return std::min<int64_t>(b * kBlockRows + wave * 32 + c, g.M - 1); };

    // ---- the rows of A
    // FUSE: where this lane's row of the stored part is (a readable stand-in, and `has` false, where there is none)
    float* arl = extra;                                             // a_r, zero beyond K
    float* dsl = extra + g.steps * kStep + wave * 32 * g.op.H;      // this wavefront's ds, [H][32]
    constexpr int kDsRegs = kMaxRowsHeads / 2;
    float dsreg[FUSE ? kDsRegs : 1];
    int rk0 = 0, rk1 = 0;
    auto rank_of = [&](int64_t b) SAR_INLINE {
        if (g.op.rank) {
            const int64_t i = row_index(b);
            rk0 = g.op.rank[i];
            rk1 = g.op.rank[i + 1];
        }
    };
    auto row_of = [&](int64_t b, bool& present) SAR_INLINE -> const float* {
        if constexpr (FUSE) {
            present = g.op.has_E && (!g.op.rank || rk1 > rk0);
            if (!g.op.has_E) return g.A;
            if (g.op.rank) return g.A + (int64_t)(present ? rk0 : 0) * g.lda;
        }
        return g.A + row_index(b) * g.lda;
    };
    auto load_ds = [&](int64_t b) SAR_INLINE {
        const int64_t first = (b * kBlockRows + wave * 32) * g.op.H, end = g.M * g.op.H;
#pragma unroll
        for (int r = 0; r < kDsRegs; ++r) {
            const int idx = lane + 64 * r;
            dsreg[r] = (g.op.ds && idx < 32 * g.op.H && first + idx < end) ? g.op.ds[first + idx] : 0.f;
        }
    };
    // kept head-major: the 32 rows of a head sit in 32 different banks
    auto keep_ds = [&]() SAR_INLINE {
#pragma unroll
        for (int r = 0; r < kDsRegs; ++r) {
            const int idx = lane + 64 * r;
            if (idx < 32 * g.op.H) dsl[(idx % g.op.H) * 32 + idx / g.op.H] = dsreg[r];
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto load_a = [&](const float* row, int step, uint4 (&a)[2]) SAR_INLINE {
        const int k = step * kStep + gq * 8;
        a[0] = load16(row + min(k, k_last));
        a[1] = load16(row + min(k + 4, k_last));
    };
    const float inv_D = FUSE ? 1.f / (float)g.op.D : 0.f;
    uint32_t low = ~0u;          // the smallest size met in this row block
    // the eight values of a step's two pieces, zero beyond K; turned: a sign bit that they take over
    auto values = [&](const uint4 (&a)[2], int step, bool has, uint32_t turned, float (&v)[8]) SAR_INLINE {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint4 av = a[p];
            const int k = step * kStep + gq * 8 + 4 * p;
            if (step == g.steps - 1) {
                if (k > k_last && rest != 0) av = front_of_piece<float>(av, rest);
                const bool beyond = k >= g.K;
                av = make_uint4(beyond ? 0u : av.x, beyond ? 0u : av.y, beyond ? 0u : av.z, beyond ? 0u : av.w);
            }
            if constexpr (FUSE) {
                if (!has) av = make_uint4(0u, 0u, 0u, 0u);
                // the piece's head, k / D, without an integer division; a_r is zero beyond K
                const int head = min((int)(((float)k + 0.5f) * inv_D), g.op.H - 1);
                const float4 ar = *reinterpret_cast<const float4*>(arl + k);
                const float r4[4] = {ar.x, ar.y, ar.z, ar.w};
                av = fuse_piece<float>(av, dsl[head * 32 + c], r4);
            }
            low = lowest(low, av);
            v[4 * p] = __uint_as_float(av.x ^ turned);
            v[4 * p + 1] = __uint_as_float(av.y ^ turned);
            v[4 * p + 2] = __uint_as_float(av.z ^ turned);
            v[4 * p + 3] = __uint_as_float(av.w ^ turned);
        }
        settle(low, v[0]);
    };

    // ---- the small operand: items of eight contraction values of one column
    // Neighbouring lanes take neighbouring memory; the second half's columns sit four apart from the first's, so that
    // two lanes of one column write to different banks.
    auto place = [](int half, int col) SAR_INLINE { return half * 32 + (col ^ (half * 4)); };
    const int item_k = (tid & 1) * 8, item_n = tid >> 1;            // (of the thread's first item; the next: 128 columns on)
    const int item_at = item_n / 32 * 192 + place(tid & 1, item_n & 31);
    uint4 bv[kPer][2];
    uint32_t low_b[kPer];        // the smallest sizes met (every row block meets the same: a test for the first one costs more)
#pragma unroll
    for (int x = 0; x < kPer; ++x) low_b[x] = ~0u;
    auto load_b = [&](int step) SAR_INLINE {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            const float* from = g.B + (int64_t)min(n0 + item_n + x * (kThreads / 2), g.N - 1) * g.K;
#pragma unroll
            for (int p = 0; p < 2; ++p) bv[x][p] = load16(from + min(step * kStep + item_k + 4 * p, k_last));
        }
    };
    // (beyond K: other values of W, which meet zeros of A)
    auto store_b = [&](int step, int buf) SAR_INLINE {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            if ((x + 1) * kThreads > NT * 64 && tid + x * kThreads >= NT * 64) break;
            float v[8];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                uint4 q = bv[x][p];
                if (rest != 0 && step * kStep + item_k + 4 * p > k_last) q = front_of_piece<float>(q, rest);
                low_b[x] = lowest(low_b[x], q);
                v[4 * p] = __uint_as_float(q.x);
                v[4 * p + 1] = __uint_as_float(q.y);
                v[4 * p + 2] = __uint_as_float(q.z);
                v[4 * p + 3] = __uint_as_float(q.w);
            }
            uint4 piece[3];
            split8(v, piece);
#pragma unroll
            for (int t = 0; t < 3; ++t) frag[buf * kBuf + item_at + x * (kThreads / 64) * 192 + t * 64] = piece[t];
        }
    };

    // ---- the results: lane holds column c; register r holds row 8 (r/4) + 4 (lane/32) + r%4
    float16_t acc[NT];
    auto clear = [&]() SAR_INLINE {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;
    };
    auto store_c = [&](int64_t b, uint32_t tiles) SAR_INLINE {      // tiles: a bit for each that is stored
        const int64_t row0 = b * kBlockRows + wave * 32 + 4 * gq;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int n = n0 + nt * 32 + c;
            if (n >= g.N || !(tiles >> nt & 1)) continue;
            float* to = g.C + row0 * g.ldc + n;
            if (row0 + 28 <= g.M) {
#pragma unroll
                for (int r = 0; r < 16; ++r) to[(int64_t)(8 * (r / 4) + (r % 4)) * g.ldc] = acc[nt][r];
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (row0 + 8 * (r / 4) + (r % 4) < g.M) to[(int64_t)(8 * (r / 4) + (r % 4)) * g.ldc] = acc[nt][r];
            }
        }
    };
    // of a row block as stored: a bit for each tile that holds an infinity or a NaN
    auto not_finite_stored = [&](int64_t b) SAR_INLINE -> uint32_t {
        const int64_t row0 = b * kBlockRows + wave * 32 + 4 * gq;
        uint32_t tiles = 0;
#pragma unroll 1
        for (int nt = 0; nt < NT; ++nt) {
            const int n = n0 + nt * 32 + c;
            float zero = 0.f;
            for (int r = 0; r < 16; ++r) {
                const int64_t i = row0 + 8 * (r / 4) + (r % 4);
                if (n < g.N && i < g.M) zero = fmaf(g.C[i * g.ldc + n], 0.f, zero);
            }
            if (__any(__builtin_isunordered(zero, zero))) tiles |= 1u << nt;
        }
        return tiles;
    };

    // ---- first loads
    const float* row;          // of the block whose steps are being fetched
    bool has = true, next_has = true;
    if constexpr (FUSE) {
        rank_of(rb);
        load_ds(rb);
    }
    row = row_of(rb, next_has);
    if constexpr (FUSE) rank_of(rb + stride);
    int64_t fetch_rb = rb;
    int fetch_step = 0;
    uint4 a[2][2];
    auto fetch = [&](uint4 (&to)[2]) SAR_INLINE {
        if (fetch_step == g.steps) {
            fetch_step = 0;
            fetch_rb += stride;
            row = row_of(fetch_rb, next_has);
            if constexpr (FUSE) {
                load_ds(fetch_rb);
                rank_of(fetch_rb + stride);
            }
        }
        load_a(row, fetch_step++, to);
    };
    load_b(0);
    fetch(a[0]);
    fetch(a[1]);
    if constexpr (FUSE) {
        for (int k = tid; k < g.steps * kStep; k += kThreads) arl[k] = g.op.ds && k < g.K ? g.op.a_r[k] : 0.f;
    }
    store_b(0, 0);
    __syncthreads();

    // ---- the steps
    int step = 0, buf = 0, ordinal = 0;
    uint64_t again = 0;      // row blocks of this wavefront to be redone (bit 63: the 64th and every later one)
    clear();
    auto turn = [&](uint4 (&cur)[2]) SAR_INLINE {
        const int after = step + 1 == g.steps ? 0 : step + 1;
        load_b(after);
        if (step == 0) {
            has = next_has;
            if constexpr (FUSE) keep_ds();
        }
        uint4 x[3];
        {
            float v[8];
            values(cur, step, has, (uint32_t)(c + step) << 31, v);
            split8(v, x);
        }
        fetch(cur);
        const uint4* fr = frag + buf * kBuf + place(gq, c);
        const float sign = step % 2 ? -1.f : 1.f;
        // A tile's 16 products are summed from zero and added to its results by vector instructions: those of two tiles
        // after the next step's values are split, of more, where registers allow, while the next tile's are multiplied.
        constexpr bool kLate = NT == 2, kAhead = !FUSE && NT > 4;
        constexpr int kSums = kLate || kAhead ? 2 : 1;
        float16_t sum[kSums];
        auto add = [&](int nt) SAR_INLINE {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float v = fmaf(r % 2 ? -sign : sign, sum[nt % kSums][r], acc[nt][r]);
                asm("" : "+v"(v));      // (or the compiler puts off the additions of every tile to the step's end)
                acc[nt][r] = v;
            }
        };
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint4 w[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] = fr[(nt * 3 + i) * 64];
            multiply_split(x, w, sum[nt % kSums]);
            if (!kLate && nt >= kSums - 1) add(nt - (kSums - 1));
            if (kAhead) __builtin_amdgcn_sched_barrier(0);
        }
        if (kAhead) add(NT - 1);
        store_b(after, buf ^ 1);
        if (kLate) {
            add(0);
            add(1);
        }
        step = after;
        if (after == 0) {
            bool redo = low < kLowBits;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) redo |= not_finite(acc[nt]);
            if (__any(redo)) again |= 1ull << min(ordinal, 63);
            low = ~0u;
            store_c(rb, ~0u);
            rb += stride;
            ++ordinal;
            clear();
        }
        __syncthreads();
        buf ^= 1;
    };
    while (true) {
        turn(a[0]);
        if (rb >= row_blocks) break;
        turn(a[1]);
        if (rb >= row_blocks) break;
    }

    // ---- tiles of 32 x 32 that are not finite or have small operands, by the fp32 instruction (any pairing of k with
    // instruction and lane group is valid as long as both operands use the same).  Which tiles these are does not depend on
    // how many of them a workgroup has: formed and stored rows give the same bits.
    int* low_cols = reinterpret_cast<int*>(split_lds);
    if (tid < NT) low_cols[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kPer; ++x)
        if (low_b[x] < kLowBits && wave + 4 * x < NT) low_cols[wave + 4 * x] = 1;
    __syncthreads();
    uint32_t tiles_b = 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tiles_b |= (uint32_t)low_cols[nt] << nt;
    tiles_b = __builtin_amdgcn_readfirstlane(tiles_b);
    if (again == 0 && tiles_b == 0) return;
    rb -= stride * ordinal;
#pragma unroll 1
    for (int o = 0; o < ordinal; ++o, rb += stride) {
        if (!(again >> min(o, 63) & 1) && tiles_b == 0) continue;
        const uint32_t tiles = tiles_b | not_finite_stored(rb);
        low = ~0u;
        clear();
        if constexpr (FUSE) {
            rank_of(rb);
            load_ds(rb);
            keep_ds();
        }
        row = row_of(rb, has);
#pragma unroll 1
        for (int s = 0; s < g.steps; ++s) {
            uint4 piece[2];
            float v[8];
            load_a(row, s, piece);
            values(piece, s, has, 0, v);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int n = min(n0 + nt * 32 + c, g.N - 1);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = s * kStep + gq * 8 + j;
                    const float w = k < g.K ? g.B[(int64_t)n * g.K + k] : 0.f;
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[j], w, acc[nt], 0, 0, 0);
                }
            }
        }
        store_c(rb, __any(low < kLowBits) ? ~0u : tiles);
    }
}

template <int NT, bool FUSE>
int launch_dx(const SplitArgs& g, hipStream_t st)
{
    size_t lds = (size_t)2 * NT * 3 * 64 * 16;
    if (FUSE) lds += ((size_t)g.steps * kStep + (size_t)(kThreads / 64) * 32 * g.op.H) * sizeof(float);
    int dev = 0, n_cu = 0;
    SAR_HIP(hipGetDevice(&dev));
    SAR_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    SAR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dx_split<NT, FUSE>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int64_t row_blocks = (g.M + kBlockRows - 1) / kBlockRows;
    const int per_cu = dx_waves(NT, FUSE);
    const int64_t resident = std::max<int64_t>(1, (int64_t)n_cu * per_cu / g.slabs);
    const int64_t groups = (std::min(row_blocks, resident) + 7) / 8;
    k_dx_split<NT, FUSE><<<(unsigned)(groups * 8 * g.slabs), kThreads, lds, st>>>(g);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// Column tiles per workgroup: at most eight (formed rows: six, by registers), the slabs as even as they come; with few
// rows fewer, so that more workgroups share the work.
int split_tiles(int64_t M, int N, int most, int* slabs)
{
    const int need = (N + 31) / 32;
    const int64_t row_blocks = (M + kBlockRows - 1) / kBlockRows;
    for (*slabs = (need + most - 1) / most;; ++*slabs) {
        int nt = (need + *slabs - 1) / *slabs;
        if (nt <= 4) nt = nt <= 2 ? 2 : 4;
        if (nt > 2 && row_blocks * *slabs < kFewWorkgroups) continue;
        *slabs = (need + nt - 1) / nt;
        return nt;
    }
}

// ---- dW = X^T dZ ---------------------------------------------------------------
//
// Both operands have the contraction index (the node) as their slow dimension.  A thread takes eight rows of four
// columns (eight 16-byte loads, a chunk ahead), splits them, and writes for each column and piece the eight rows as one
// 16-byte unit to LDS: the transposed fragment, which the wavefronts read with one access per lane.  A unit's column is
// exchanged within its group of four (column ^ (column / 8 % 4)), which puts the columns 4q + j of neighbouring lanes
// and the neighbouring columns of a read alike on different banks.  One workgroup of eight wavefronts per CU; the output
// tile is 128 x NW, 32 or 64 rows a chunk, double buffered, one barrier per chunk.  Rows are split into slabs over the grid;
// k_sum_slabs adds the partial tiles in a fixed order.
//
// The matrix cores cut a product's bits below the sum's instead of rounding them, always downwards: five small terms
// added to a long sum every 16 rows made an error of one sign that the slabs' sums kept (a million rows, 64 x 64: 2.4e-6
// of the result, the fp32 instruction 5.8e-7).  So a chunk's 32 rows are summed by themselves, all small terms before the
// large ones, and the chunk's sum is added to the slab's by vector instructions, which round to nearest; and every other
// chunk's X is taken with the other sign and its sum subtracted, so that what is cut falls on either side.  Error of dW
// against 64-bit sums, fp32 instruction and here: 306250 rows 256 x 256 6.3e-7 / 1.9e-7, 2450000 rows 400 x 400 3.5e-6 /
// 6.3e-7, 4096 rows 64 x 64 1.3e-7 / 0.9e-7, 1000 rows 100 x 256 2.2e-7 / 0.8e-7; 64 x 64 of 1, 2, 3, 4, 8 rows 2.5e-8 / 3.5e-8,
// 3.1e-8 / 3.4e-8, 3.9e-8 / 3.2e-8, 4.1e-8 / 3.2e-8, 4.8e-8 / 3.1e-8: a product's last addition is cut and not rounded, so one or
// two rows stay with the fp32 instruction.  (A result whose other products are zeros is as far off as one of one row.)
//
// A chunk is on its way while the one before it is split and the one before that is multiplied.  Of the two wavefronts
// of a SIMD one splits before it multiplies and the other after, so that the vector instructions of one run beside the
// matrix instructions of the other.  Measured against the fp32 instruction, plain / with formed rows, us: 306250 rows 100
// x 256 186 / 209 -> 136 / 145, 256 x 256 351 / 391 -> 259 / 267; 2450000 rows 400 x 400 10740 -> 6950; 8000 rows 256 x
// 256 35 / 41 -> 23 / 26; 4096 rows 64 x 64 10.1 / 11.0 -> 8.6 / 10.5.  Bound by the chunk's latency and, in wide products,
// by issue: matrix instructions take 41 to 52% of the cycles, vector instructions 45 to 47%, at 1.7 to 1.9 GHz.
constexpr int kDwThreads = 512;
constexpr int kDwSum = 32;           // rows summed by themselves
constexpr int kDwKf = 128;
// Rows of a chunk.  The narrow tile takes twice as many: with 32 one workgroup per CU (formed rows, by registers) had 16 KB
// on their way and waited for them (1000000 rows 64 x 64 formed 307 -> 158 us, stored, two workgroups per CU, 129 -> 137; 40000
// rows 128 x 64 21.2 -> 18.8 and 18.7 -> 17.2).
constexpr int dw_rows(int nw) { return nw == 64 ? 64 : 32; }

template <bool FUSE, int NW, bool RAG>
__global__ __launch_bounds__(kDwThreads, 2) void k_dw_split(const float* __restrict__ X, const float* __restrict__ dZ,
                                                            RowsOp op, float* __restrict__ partial, int64_t M, int K,
                                                            int N, int64_t rows_per_slab)
{
    static_assert(!(FUSE && RAG), "");
    constexpr int kNt = NW == 64 ? 1 : 2;     // tiles of 32 columns per wavefront
    constexpr int kCols = NW / 32 / kNt;      // wavefronts side by side
    constexpr int kKg = 8 / kCols;            // groups of kf-tiles
    constexpr int kKt = 4 / kKg;              // kf-tiles per wavefront
    constexpr int kRows = dw_rows(NW), kOct = kRows / 8;
    constexpr int kPlane = kOct * (kDwKf + NW);           // units of one piece of a chunk
    constexpr int kBuf = 3 * kPlane;
    extern __shared__ __attribute__((aligned(16))) uint4 dw_lds[];
    __shared__ int redo;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, gq = lane >> 5;
    const int kf0 = blockIdx.z * kDwKf, n0 = blockIdx.y * NW;
    const int64_t m_beg = (int64_t)blockIdx.x * rows_per_slab;
    const int64_t m_end = std::min<int64_t>(M, m_beg + rows_per_slab);
    const int cw = wave % kCols, kg = wave / kCols;
    // this wavefront's tiles that exist (its kf-tile kt is the workgroup's kt * kKg + kg)
    const int kt_n = max(0, min(kKt, ((K - kf0 + 31) / 32 + kKg - 1 - kg) / kKg));
    const bool some = kt_n > 0 && n0 + 32 * kNt * cw < N;

    // ---- staging: which eight rows of which four columns are this thread's
    // (whole wavefronts: the branches on it are uniform)
    constexpr int kOfDz = NW / 4 * kOct, kOfX = kDwKf / 4 * kOct;
    static_assert(kOfDz % 64 == 0 && kOfDz + kOfX <= kDwThreads, "");
    const bool of_dz = wave * 64 < kOfDz, of_x = !of_dz && wave * 64 < kOfDz + kOfX;
    const int u = of_dz ? tid : tid - kOfDz, quads = of_dz ? NW / 4 : kDwKf / 4;
    const int oct = u / quads, col = 4 * (u % quads);
    const int width = of_dz ? N : K, first = (of_dz ? n0 : kf0) + col;
    // (columns beyond the width are another column's values: nothing of them is stored)
    const int from_col = max(0, min(first, width - 4));
    const float* base = (of_dz ? dZ : X) + from_col;
    const int unit0 = oct * (kDwKf + NW) + (of_dz ? kDwKf + col : col);
    const int head = FUSE ? min(first, N - 4) / op.D : 0;
    const bool formed = FUSE && of_dz;
    uint4 ahead[8] = {};
    // FUSE: the lanes that share eight rows load their nine entries of the row map one each, a chunk ahead of the rows,
    // and their ds in turn, kShare (row, head) at a time; what a lane needs it takes from the others
    constexpr int kShare = std::min(64, NW / 4);
    constexpr int kDsOwn = FUSE ? 8 * kMaxRowsHeads / kShare : 1;
    const int rank_in = lane % kShare, share0 = lane - rank_in;
    int map = 0, absent = 0;      // absent: a bit for each of the eight rows that E does not have
    float ds_own[kDsOwn] = {}, ar[4];
    if constexpr (FUSE)
#pragma unroll
        for (int x = 0; x < 4; ++x) ar[x] = formed && op.ds ? op.a_r[from_col + x] : 0.f;
    auto fetch_rank = [&](int64_t m0) SAR_INLINE {
        if constexpr (FUSE) {
            if (formed && op.rank) map = op.rank[std::min<int64_t>(m0 + 8 * oct + min(rank_in, 8), M)];
        }
    };
    auto from_lane = [&](auto v, int of) SAR_INLINE {
        // (one group: the lane's number is the same for all)
        return kShare == 64 ? __builtin_bit_cast(decltype(v), __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), of))
                            : __shfl(v, share0 + of);
    };
    auto load_row = [&](const float* row) SAR_INLINE -> uint4 {
        if constexpr (RAG) {
            if (width < 4) {
                float v[4] = {};
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (x < width) v[x] = row[x];
                return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                                  __float_as_uint(v[3]));
            }
        }
        return load16(row);
    };
    auto fetch = [&](int64_t m0) SAR_INLINE {
        if (of_dz || of_x) {
            const int64_t m = m0 + 8 * oct;
            int64_t from[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) from[j] = std::min<int64_t>(m + j, M - 1);   // (beyond: zeroed when they are split)
            if constexpr (FUSE) {
                if (formed) {
                    if (op.ds) {
                        const float* of_row = op.ds + std::min<int64_t>(m + rank_in % 8, M - 1) * op.H;
#pragma unroll
                        for (int i = 0; i < kDsOwn; ++i)
                            if (i == 0 || i * (kShare / 8) < op.H)
                                ds_own[i] = of_row[min(i * (kShare / 8) + rank_in / 8, op.H - 1)];
                    }
                    if (op.rank) {
                        int rk[9];
#pragma unroll
                        for (int j = 0; j < 9; ++j) rk[j] = from_lane(map, j);
                        absent = 0;
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            absent |= rk[j + 1] > rk[j] ? 0 : 1 << j;
                            from[j] = rk[j + 1] > rk[j] ? rk[j] : 0;
                        }
                    }
                    if (!op.has_E) {      // (a stand-in of one row)
                        absent = 255;
#pragma unroll
                        for (int j = 0; j < 8; ++j) from[j] = 0;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) ahead[j] = load_row(base + from[j] * width);
        }
        fetch_rank(m0 + kRows);
    };
    uint32_t low = ~0u;           // the smallest size this thread has split
    auto commit = [&](int64_t m0, int buf, auto keep) SAR_INLINE {
        if (!(of_dz || of_x)) return;
        constexpr bool KEEP = decltype(keep)::value;
        // every other 32 rows with the sign of X turned over (see above)
        const float sign = of_x && ((m0 + 8 * oct) & kDwSum) ? -1.f : 1.f;
        float dsv[FUSE ? 8 : 1] = {};
        if constexpr (FUSE) {
            if (formed && op.ds) {
#pragma unroll
                for (int i = 0; i < kDsOwn; ++i) {
                    if (i > 0 && i * (kShare / 8) >= op.H) break;
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float v = __shfl(ds_own[i], share0 + head * 8 % kShare + j);
                        dsv[j] = i == 0 || head / (kShare / 8) == i ? v : dsv[j];
                    }
                }
            }
        }
        float v[4][8];
        const int64_t left = m_end - (m0 + 8 * oct);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            uint4 r = ahead[j];
            if constexpr (RAG) {
                if (width > 4 && first < width && first + 4 > width) r = front_of_piece<float>(r, width % 4);
            }
            if constexpr (FUSE) {
                if (absent >> j & 1) r = make_uint4(0u, 0u, 0u, 0u);
                if (formed) r = fuse_piece<float>(r, dsv[j], ar);
            }
            if constexpr (!KEEP) low = lowest(low, r);
            v[0][j] = sign * __uint_as_float(r.x);
            v[1][j] = sign * __uint_as_float(r.y);
            v[2][j] = sign * __uint_as_float(r.z);
            v[3][j] = sign * __uint_as_float(r.w);
        }
        settle(low, v[0][0]);
        if (left < 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int x = 0; x < 4; ++x) v[x][j] = j < left ? v[x][j] : 0.f;
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            // (KEEP: the eight values themselves, in the places of the first two pieces)
            uint4 piece[3];
            if constexpr (KEEP) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    piece[t] = make_uint4(__float_as_uint(v[x][4 * t]), __float_as_uint(v[x][4 * t + 1]),
                                          __float_as_uint(v[x][4 * t + 2]), __float_as_uint(v[x][4 * t + 3]));
            } else {
                split8(v[x], piece);
            }
#pragma unroll
            for (int t = 0; t < (KEEP ? 2 : 3); ++t)
                dw_lds[buf * kBuf + t * kPlane + unit0 + (x ^ (col >> 3 & 3))] = piece[t];
        }
    };

    float16_t acc[kKt][kNt];
    const int swap = c >> 3 & 3;              // (a tile's first column is a multiple of 32)
    auto fragment = [&](int buf, int step, int at, uint4 (&w)[3]) SAR_INLINE {
        const uint4* p = dw_lds + buf * kBuf + (2 * step + gq) * (kDwKf + NW) + at + (c ^ swap);
#pragma unroll
        for (int t = 0; t < 3; ++t) w[t] = p[t * kPlane];
    };
    auto multiply_32 = [&](int buf, int first, float sign, auto keep) SAR_INLINE {      // from the chunk's step `first` on
        uint4 b[kNt][2][3];
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
            for (int s = 0; s < 2; ++s) fragment(buf, first + s, kDwKf + 32 * (kNt * cw + nt), b[nt][s]);
#pragma unroll
        for (int kt = 0; kt < kKt; ++kt) {
            if (kt >= kt_n) break;
            uint4 a[2][3];
#pragma unroll
            for (int s = 0; s < 2; ++s) fragment(buf, first + s, 32 * (kt * kKg + kg), a[s]);
            float16_t sum[kNt] = {};
            if constexpr (decltype(keep)::value) {
#pragma unroll
                for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const uint4 x = a[s][t], y = b[nt][s][t];
                            const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                sum[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(xs[j]),
                                                                               __uint_as_float(ys[j]), sum[nt], 0, 0, 0);
                        }
            } else {
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int nt = 0; nt < kNt; ++nt)
                            sum[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8_t, a[s][kTerm[t][0]]),
                                __builtin_bit_cast(bf16x8_t, b[nt][s][kTerm[t][1]]), sum[nt], 0, 0, 0);
            }
#pragma unroll
            for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[kt][nt][r] = fmaf(sign, sum[nt][r], acc[kt][nt][r]);
        }
    };
    auto multiply = [&](int buf, int64_t m0, auto keep) SAR_INLINE {
        if (!some) return;
#pragma unroll
        for (int part = 0; part < kRows / kDwSum; ++part)
            multiply_32(buf, 2 * part, (m0 + part * kDwSum) & kDwSum ? -1.f : 1.f, keep);
    };
    auto slab = [&](auto keep) SAR_INLINE {
#pragma unroll
        for (int x = 0; x < kKt; ++x)
#pragma unroll
            for (int y = 0; y < kNt; ++y)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
        if (m_beg < m_end) {
            fetch_rank(m_beg);
            fetch(m_beg);
            commit(m_beg, 0, keep);
            fetch(m_beg + kRows);
        }
        __syncthreads();
        int buf = 0;
        for (int64_t m0 = m_beg; m0 < m_end; m0 += kRows, buf ^= 1) {
            auto stage = [&]() SAR_INLINE {
                if (m0 + kRows < m_end) {
                    commit(m0 + kRows, buf ^ 1, keep);
                    fetch(m0 + 2 * kRows);         // (beyond the end: the last row, used by nobody)
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // (of a SIMD's two wavefronts one splits first, the other multiplies first)
            if (wave < kDwThreads / 128) stage();
            multiply(buf, m0, keep);
            if (wave >= kDwThreads / 128) stage();
            __syncthreads();
        }
    };
    // (sums of one or two products: closer by the fp32 instruction, see above)
    if (M > 2) slab(std::false_type{});
    bool again = M <= 2 || low < kLowBits;
#pragma unroll
    for (int x = 0; x < kKt; ++x)
#pragma unroll
        for (int y = 0; y < kNt; ++y) again |= not_finite(acc[x][y]);
    if (tid == 0) redo = 0;
    __syncthreads();
    if (again) redo = 1;
    __syncthreads();
    if (redo) slab(std::true_type{});

    // lane holds column c; register r holds row 8 (r/4) + 4 (lane/32) + r%4
    float* out = partial + (int64_t)blockIdx.x * K * N;
#pragma unroll
    for (int kt = 0; kt < kKt; ++kt)
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt) {
            const int n = n0 + 32 * (kNt * cw + nt) + c;
            if (n >= N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kf = kf0 + 32 * (kt * kKg + kg) + 8 * (r / 4) + 4 * gq + (r % 4);
                if (kf < K) out[(int64_t)kf * N + n] = acc[kt][nt][r];
            }
        }
}

template <bool FUSE, int NW, bool RAG>
int launch_dw(const float* X, const float* dZ, const RowsOp& op, float* partial, int64_t n, int K, int F, int slabs,
              int64_t rows_per_slab, hipStream_t st)
{
    constexpr size_t lds = (size_t)2 * 3 * (dw_rows(NW) / 8) * (kDwKf + NW) * 16;
    SAR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dw_split<FUSE, NW, RAG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const dim3 grid((unsigned)slabs, (unsigned)((F + NW - 1) / NW), (unsigned)((K + kDwKf - 1) / kDwKf));
    k_dw_split<FUSE, NW, RAG><<<grid, kDwThreads, lds, st>>>(X, dZ, op, partial, n, K, F, rows_per_slab);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

}  // namespace

namespace sar {

int split_dx(const float* dZ, const RowsOp* op, const float* W, float* dX, int64_t n, int K, int F, hipStream_t st)
{
    SplitArgs g{dZ, F, n, W, dX, K, F, K, (F + kStep - 1) / kStep, 0, op ? *op : RowsOp{}};
    // (the second step is fetched before the first is multiplied: of the same rows)
    if (g.steps < 2) return sar::fail(SAR_ERR_STATE, "the split product for dX takes more than %d columns", kStep);
    const int nt = split_tiles(n, K, op ? 6 : 8, &g.slabs);
    auto with = [&](auto fuse) {
        constexpr bool FUSE = decltype(fuse)::value;
        switch (nt) {
            case 2: return launch_dx<2, FUSE>(g, st);
            case 4: return launch_dx<4, FUSE>(g, st);
            case 5: return launch_dx<5, FUSE>(g, st);
            case 6: return launch_dx<6, FUSE>(g, st);
        }
        if constexpr (!FUSE) return nt == 7 ? launch_dx<7, false>(g, st) : launch_dx<8, false>(g, st);
        return sar::fail(SAR_ERR_STATE, "formed rows take at most six column tiles");
    };
    return op ? with(std::true_type{}) : with(std::false_type{});
}

int split_dw(const float* X, const float* dZ, const RowsOp* op, float* partial, int64_t n, int K, int F, int most_slabs,
             int* slabs, hipStream_t st)
{
    const int nw = F <= 64 ? 64 : F <= 128 ? 128 : 256;
    const int64_t tiles = (int64_t)((F + nw - 1) / nw) * ((K + kDwKf - 1) / kDwKf);
    // As many workgroups as run at once, one per CU, where all have the same work and where output tiles are narrow; where the
    // last of wider tiles are narrower twice as many, so that CUs that end early take another.  (Each writes a partial tile:
    // 100000 rows 283 x 100 104 us with 341 slabs, 94 with 170; 40000 rows 203 x 64 30 with 512 over both tiles, 22 with 256,
    // 250000 rows 94 and 87.)  Stored and formed rows alike: their sums are to be the same bits.
    const bool even = (F % nw == 0 || F <= nw) && (K % kDwKf == 0 || K <= kDwKf);
    const int64_t want = std::max<int64_t>(1, (even || nw == 64 ? 256 : 512) / tiles);
    *slabs = (int)std::min<int64_t>(want, most_slabs);
    const int64_t rows = ((n + *slabs - 1) / *slabs + kDwSum - 1) / kDwSum * kDwSum;
    auto with = [&](auto fuse, auto ragged) {
        constexpr bool FUSE = decltype(fuse)::value, RAG = decltype(ragged)::value;
        const RowsOp o = op ? *op : RowsOp{};
        if (nw == 64) return launch_dw<FUSE, 64, RAG>(X, dZ, o, partial, n, K, F, *slabs, rows, st);
        if (nw == 128) return launch_dw<FUSE, 128, RAG>(X, dZ, o, partial, n, K, F, *slabs, rows, st);
        return launch_dw<FUSE, 256, RAG>(X, dZ, o, partial, n, K, F, *slabs, rows, st);
    };
    if (op) return with(std::true_type{}, std::false_type{});    // (whole pieces)
    if (K % 4 == 0 && F % 4 == 0) return with(std::false_type{}, std::false_type{});
    return with(std::false_type{}, std::true_type{});
}

}  // namespace sar
