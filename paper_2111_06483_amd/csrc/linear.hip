// The dense node-wise transform of Eq. 1 (z = W h, row-major Z = X W) and its
// backward (what Z.backward(E) does in Alg. 2: dW = X^T dZ, dX = dZ W^T) on the
// gfx950 matrix cores.  This is the one real contraction on the path.
//
// fp32 rows are multiplied with V_MFMA_F32_32X32X2_F32 (fp32 in, fp32 accumulate) in the forward
// product, whose last bits decide slopes and signs further on; the two products of the backward pass
// go through the bf16 matrix cores in three pieces per value, which is both faster and closer to the
// exact sums (linear_split.hip).  bf16-stored rows go through V_MFMA_F32_32X32X16_BF16:
// the products are exact there, and the fp32 weight matrix is split into two bf16 terms,
// W = hi + lo (+ an error below 2^-17 |W|), multiplied in two instructions, which is far
// below the bf16 rounding of the stored result.
//
// Z = X W and dX = dZ W^T read their rows straight into registers.  Where the small operand
// fits in LDS it stays there (k_gemm_skinny); where it does not it passes through LDS in
// steps of the contraction (k_gemm_steps).  dW of bf16 rows has a kernel of its own (k_dw).  Few rows
// go another way (linear_few.hip).
#include <algorithm>

#include "linear_common.h"
#include "linear_few.h"
#include "linear_split.h"
#include "sar_internal.h"

namespace {

using namespace sar;

// ---- skinny products: the small operand resident in LDS --------------------
//
// In Z = X W and dX = dZ W^T the left operand has millions of rows whose
// contraction index is contiguous in memory, which is exactly what an MFMA A
// fragment wants from a lane: lane l of a 32-row tile supplies row l%32 and a
// 16-byte piece of it (4 floats or 8 bf16 values) chosen by l/32.  So the big
// operand goes from HBM straight into registers, never through LDS.  The small
// operand (at most a few hundred KB) is laid out in LDS once per workgroup, in
// the order the B fragments are consumed: one 16-byte unit per lane, 64 units
// per fragment, so every ds_read_b128 is conflict-free.  After that one
// barrier the wavefronts never synchronise again: each walks over its own
// 32-row tiles, keeping NT 32x32 accumulators (32 x NT*32 outputs) in
// registers and two pairs of 16-byte pieces of its rows, one in flight while the other is used.
//
// fp32: a chunk is 8 contraction values; lane group g = l/32 holds values
//       8t+4g .. 8t+4g+3, consumed by four V_MFMA_F32_32X32X2_F32 (whose A and
//       B operands both take "their k" from the lane group, so any pairing of
//       k with (step, group) is valid as long as both operands use the same).
// bf16: a chunk is 16 values, one V_MFMA_F32_32X32X16_BF16 per bf16 half of the
//       fp32 small operand (hi and lo).

constexpr int kSkinnyWaves = 8;
constexpr int kSkinnyThreads = 64 * kSkinnyWaves;
constexpr size_t kSkinnyMaxLds = 160 * 1024;   // all of a CU's LDS: one workgroup per CU then

struct SkinnyArgs {
    const void* A;     // [M, K], row stride lda, contraction index contiguous
    int64_t lda, M;
    const float* B;    // B(k, n) = B[k * sbk + n * sbn]
    int64_t sbk, sbn;
    void* C;           // [M, N], row stride ldc
    int64_t ldc;
    int K, N;
    int chunks;        // ceil(K / chunk length)
    // score projections (Eq. 3: the two halves of a^T (z_i || z_j)) as one more
    // accumulator tile: column h of it is x . (W_h a1_h), column H+h is x . (W_h a2_h)
    const float* a1;   // [H, D] or null
    const float* a2;
    float* s1;         // [M, H] or null
    float* s2;
    int H, D;
    // byte offset in LDS of the per-wavefront 32 x 32 staging tiles through which the outputs
    // are stored as whole 64- or 128-byte row segments, or 0 to store element-wise
    int stage_off;
    RowsOp op;         // FUSE only: how the rows of A are formed
    int vec_off = 0;   // Scores::kRows: byte offset in LDS of the columns' values of a1 and of a2
};

// kTile: as one more accumulator tile, from the unrounded sums.  kRows: from the rows as they are stored.
enum class Scores { kNone, kTile, kRows };


// Sums over lanes of four, the same bits in each.
__device__ inline float add_xor2(float v)
{
    return v + __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x4E /* lane ^ 2 */, 0xf, 0xf, true));
}
__device__ inline float quad_sum(float v)
{
    return add_xor2(v + __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0xB1 /* lane ^ 1 */, 0xf, 0xf, true)));
}

// FUSE: the rows of A are not stored; each piece is formed where it is multiplied (RowsOp, K <= 256).
// Between the epilogues a wavefront's staging tile is idle, so it holds what the pieces need: the
// tile's 32 x H values of ds and the K values of a_r.  The row map and ds of a tile are read one
// tile ahead (the map two), like the first pieces of its rows.
constexpr int kDsRegs = 8;   // 32 rows x H <= 16 heads of ds, 64 lanes

// Scores::kRows (bf16, heads of 32, 64 or 128 values): on their way through the staging tile four lanes hold a row's 32
// values of a tile, eight each, as they would in a pass over the stored rows (k_scores in gat.hip).  They form the same sums in
// the same order (a head's tiles are added pairwise, as that pass adds its lanes), so the bits are those of that pass.
//
// RAG: K is no whole number of pieces.
template <typename TA, typename TC, int NT, Scores S, bool FUSE, bool RAG>
__global__ __launch_bounds__(kSkinnyThreads) void k_gemm_skinny(SkinnyArgs g)
{
    constexpr bool SC = S == Scores::kTile, SR = S == Scores::kRows;
    static_assert(!((SC || SR) && FUSE), "the fused operand is that of dX = E W^T, which has no scores");
    static_assert(!(RAG && (FUSE || SC)), "");
    static_assert(!SR || sizeof(TC) == 2, "");
    constexpr int NA = NT + (SC ? 1 : 0);   // accumulator tiles: NT of the product, one of scores
    extern __shared__ __attribute__((aligned(16))) unsigned char skinny_lds[];
    constexpr bool BF = sizeof(TA) == 2;
    constexpr int kChunk = BF ? 16 : 8;
    constexpr int kFragsPerTile = BF ? 2 : 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, gq = lane >> 5;
    const int64_t n0 = (int64_t)blockIdx.y * (NT * 32);
    uint4* frag = reinterpret_cast<uint4*>(skinny_lds);

    const TA* A = static_cast<const TA*>(g.A);
    const int64_t n_tiles = (g.M + 31) / 32;
    // a few tiles spread over the workgroups before they fill one
    const int64_t stride = (int64_t)gridDim.x * kSkinnyWaves;
    int64_t tile = (int64_t)blockIdx.x + (int64_t)gridDim.x * wave;

    // The first pieces of the first tile travel while the small operand is staged.
    //
    // Loads are unconditional (a piece that would end beyond the row is read from the row's last 16
    // bytes; what of it is beyond, or the piece before it carries as well, is zeroed where it is used)
    // and the main loop below is straight-line code, so that the compiler can count the
    // loads in flight and wait for the oldest only; with branches around them it waits for all of
    // them at every chunk, which leaves the ring no depth.
    const int k_last = g.K - kChunk / 2;
    auto load_piece = [&](const TA* rowp, int t) -> uint4 {
        const int k = t * kChunk + gq * (kChunk / 2);
        return load16(rowp + min(k, k_last));
    };
    // a piece that starts at k_first < K and was read from k_last < k_first: its values move to the front
    const int rest = g.K % (kChunk / 2);
    auto row_ptr = [&](int64_t tl) { return A + std::min<int64_t>(tl * 32 + c, g.M - 1) * g.lda; };

    // FUSE: where this lane's row of the stored part is (row 0, and `has` false, where there is none:
    // the loads stay unconditional), the tile's ds values on their way to LDS, the lane's four a_r
    float* dsl = nullptr;
    float* arl = nullptr;
    float arreg[4] = {0.f, 0.f, 0.f, 0.f}, dsreg[kDsRegs];
    int nrk0 = 0, nrk1 = 0;
    bool has = false;
    const float inv_D = FUSE ? 1.f / (float)g.op.D : 0.f;
    auto rank_of = [&](int64_t tl, int& r0, int& r1) {
        if (g.op.rank && tl < n_tiles) {
            const int64_t i = std::min<int64_t>(tl * 32 + c, g.M - 1);
            r0 = g.op.rank[i];
            r1 = g.op.rank[i + 1];
        }
    };
    auto row_ptr_fused = [&](int64_t tl, int r0, int r1, bool& present) -> const TA* {
        if (!g.op.has_E) {
            present = false;
            return A;                      // a readable stand-in row
        }
        if (g.op.rank) {
            present = r1 > r0;
            return A + (int64_t)(present ? r0 : 0) * g.lda;
        }
        present = true;
        return row_ptr(tl);
    };
    auto load_ds = [&](int64_t tl) {
        const int64_t first = tl * 32 * g.op.H, end = g.M * g.op.H;
#pragma unroll
        for (int r = 0; r < kDsRegs; ++r) {
            const int idx = lane + 64 * r;
            dsreg[r] = (g.op.ds && idx < 32 * g.op.H && first + idx < end) ? g.op.ds[first + idx] : 0.f;
        }
    };
    if constexpr (FUSE) {
        dsl = reinterpret_cast<float*>(skinny_lds + g.stage_off + wave * (32 * 32 * (int)sizeof(TC)));
        arl = dsl + 32 * g.op.H;
    }

    // Two sets of pieces: while the chunks of one set are multiplied, the other set travels.
    // The loads of a set are issued together, ahead of the other set's MFMAs, and are first
    // needed a whole set later.  (The compiler waits for every load in flight, not for the oldest,
    // wherever stores may be in flight too, so a deeper ring of single loads gains nothing.)
    // chunks per set: about 2000 MFMA cycles of one wavefront either way (two where registers run out: with four and scores of
    // the stored rows four are spilled, 3.5 M rows of 128 to 256 712 us instead of 696)
    constexpr int PS = (BF && !((SC || SR) && NT == 8)) ? 4 : 2;
    uint4 a[PS], b[PS];
    const TA* rowp;
    if constexpr (FUSE) {
        rank_of(tile, nrk0, nrk1);
        rowp = row_ptr_fused(tile, nrk0, nrk1, has);
        if (tile < n_tiles) load_ds(tile);
        rank_of(tile + stride, nrk0, nrk1);
    } else {
        rowp = row_ptr(tile);
    }
#pragma unroll
    for (int u = 0; u < PS; ++u) a[u] = load_piece(rowp, u);
    // Staging is one long wait of a step of few nodes, so its loads travel together, eight units'
    // worth per thread and round: unconditional (values beyond K or N are read from the last row or
    // column and dropped), and along the contraction by 16 bytes where that is the contiguous direction.
    // bf16: a thread makes the hi and the lo unit of the same eight values.  (bf16, whole kernel, before:
    // loads behind a branch each, and every value twice: 254 x 200 over 30000 rows 46 -> 19..25 us, 219 x 36
    // over 14000 rows 32 -> 13 us.)
    const int units = g.chunks * NA * 64;
    constexpr int kVals = kChunk / 2, kRound = 32 / kVals;
    for (int u0 = tid; u0 < units; u0 += kRound * kSkinnyThreads) {
        float val[kRound][kVals];
        auto where = [&](int u, int& kb, int64_t& n) {
            const int f = u >> 6, nt = f % NA, t = f / NA;
            // the score tile starts as zeros; its entries are written below
            n = (SC && nt == NT) ? g.N : n0 + nt * 32 + (u & 31);
            kb = t * kChunk + ((u & 63) >> 5) * kVals;
        };
#pragma unroll
        for (int x = 0; x < kRound; ++x) {
            int kb;
            int64_t n;
            where(min(u0 + x * kSkinnyThreads, units - 1), kb, n);
            const float* from = g.B + std::min<int64_t>(n, g.N - 1) * g.sbn;
            if (!RAG && g.sbk == 1) {
                // (K is a whole number of pieces, so a piece lies inside the row or beyond it)
#pragma unroll
                for (int j = 0; j < kVals; j += 4) {
                    const uint4 v = load16(from + min(kb, g.K - kVals) + j);
                    val[x][j] = __uint_as_float(v.x);
                    val[x][j + 1] = __uint_as_float(v.y);
                    val[x][j + 2] = __uint_as_float(v.z);
                    val[x][j + 3] = __uint_as_float(v.w);
                }
            } else {
#pragma unroll
                for (int j = 0; j < kVals; ++j) val[x][j] = from[(int64_t)min(kb + j, g.K - 1) * g.sbk];
            }
        }
#pragma unroll
        for (int x = 0; x < kRound; ++x) {
            const int u = u0 + x * kSkinnyThreads;
            if (u >= units) break;
            int kb;
            int64_t n;
            where(u, kb, n);
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < kVals; ++j) {
                const float v = (kb + j < g.K && n < g.N) ? val[x][j] : 0.f;
                if (!BF) {
                    hi[j % 4] = __float_as_uint(v);
                } else {
                    const uint32_t h = f32_to_bf16_rne(v), l = f32_to_bf16_rne(v - __uint_as_float(h << 16));
                    hi[j / 2] = (j & 1) ? hi[j / 2] | (h << 16) : h;
                    lo[j / 2] = (j & 1) ? lo[j / 2] | (l << 16) : l;
                }
            }
            if (!BF) {
                frag[u] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            } else {
                uint4* at = frag + (u >> 6) * 128 + (u & 63);
                at[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                at[64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
        }
    }
    if (SC) {
        // (W a)[k][h] = sum_d W[k][h*D + d] a[h][d]: z_h . a_h = x . (W_h a_h), so the scores
        // are 2H more output columns of the same product, taken from the unrounded sums
        __syncthreads();
        // a head's two score columns belong to the column slab that holds the head's first
        // column; the other slabs leave them at zero and do not store them
        const int cols = 2 * g.H;
        for (int p = tid; p < g.K * cols; p += kSkinnyThreads) {
            const int k = p / cols, col = p % cols;
            const int h = col < g.H ? col : col - g.H;
            const float* av = col < g.H ? g.a1 : g.a2;
            const int t = k / kChunk, gk = (k / (kChunk / 2)) & 1, e = k % (kChunk / 2);
            float v = 0.f;
            if (av && (h * g.D) / (NT * 32) == (int)blockIdx.y) {
                if (!BF && (int64_t)(h + 1) * g.D <= n0 + NT * 32) {
                    // this head's part of row k of W is in LDS already (exact fp32 values, fragment
                    // order): D strided reads of global memory per product would cost more than
                    // the whole staging
                    const float* wk = reinterpret_cast<const float*>(frag) + ((size_t)t * NA * 64 + gk * 32) * 4 + e;
#pragma unroll 8
                    for (int d = 0; d < g.D; ++d) {
                        const int n = h * g.D + d - (int)n0;
                        v = fmaf(wk[((n >> 5) * 64 + (n & 31)) * 4], av[h * g.D + d], v);
                    }
                } else {
                    const float* wrow = g.B + (int64_t)k * g.sbk + (int64_t)h * g.D * g.sbn;
                    for (int d = 0; d < g.D; ++d) v = fmaf(wrow[d * g.sbn], av[h * g.D + d], v);
                }
            }
            if (!BF) {
                reinterpret_cast<float*>(frag)[(((size_t)t * NA + NT) * 64 + gk * 32 + col) * 4 + e] = v;
            } else {
                uint16_t* fh = reinterpret_cast<uint16_t*>(frag);
                const uint32_t hi = f32_to_bf16_rne(v);
                const size_t at = ((size_t)t * NA + NT) * 2 * 64 + gk * 32 + col;
                fh[at * 8 + e] = (uint16_t)hi;
                fh[(at + 64) * 8 + e] = (uint16_t)f32_to_bf16_rne(v - __uint_as_float(hi << 16));
            }
        }
    }
    float* const vecs = reinterpret_cast<float*>(skinny_lds + g.vec_off);
    if constexpr (SR) {
        for (int x = tid; x < 2 * NT * 32; x += kSkinnyThreads) {
            const float* const from = x < NT * 32 ? g.a1 : g.a2;
            const int64_t n = n0 + x % (NT * 32);
            vecs[x] = from && n < g.N ? from[n] : 0.f;
        }
    }
    __syncthreads();

    if (tile >= n_tiles) return;
    if constexpr (FUSE) {
#pragma unroll
        for (int x = 0; x < 4; ++x) arreg[x] = (g.op.ds && lane * 4 + x < g.K) ? g.op.a_r[lane * 4 + x] : 0.f;
    }
    // the last chunk, where K may end, is always one of the last chunks below
    const int full = (g.chunks - 1) / (2 * PS) * (2 * PS);

    for (; tile < n_tiles; tile += stride) {
        float16_t acc[NA];
#pragma unroll
        for (int nt = 0; nt < NA; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;
        if constexpr (FUSE) {
            // the previous tile's outputs have left the staging tile
            // kept head-major, [H][32 rows]: the 32 rows of a head sit in 32 different banks
#pragma unroll
            for (int r = 0; r < kDsRegs; ++r) {
                const int idx = lane + 64 * r;
                if (idx < 32 * g.op.H) dsl[(idx % g.op.H) * 32 + idx / g.op.H] = dsreg[r];
            }
            *reinterpret_cast<float4*>(arl + lane * 4) = make_float4(arreg[0], arreg[1], arreg[2], arreg[3]);
            __builtin_amdgcn_wave_barrier();
        }

        auto multiply = [&](const uint4& piece, int t, auto last) {
            const int k_first = t * kChunk + gq * (kChunk / 2);
            uint4 av = piece;
            if constexpr (decltype(last)::value) {
                const bool beyond = k_first >= g.K;
                if constexpr (RAG)
                    if (k_first > k_last) av = front_of_piece<TA>(av, rest);
                av = make_uint4(beyond ? 0u : av.x, beyond ? 0u : av.y, beyond ? 0u : av.z, beyond ? 0u : av.w);
            }
            if constexpr (FUSE) {
                if (!has) av = make_uint4(0u, 0u, 0u, 0u);
                // a_r is zero beyond K, so a piece beyond the row stays zero
                // head of the piece: k_first / D for 0 <= k_first < 512, without an integer division
                const int head = min((int)(((float)k_first + 0.5f) * inv_D), g.op.H - 1);
                const float d = dsl[head * 32 + c];
                float ar[kChunk / 2];
#pragma unroll
                for (int x = 0; x < kChunk / 2; x += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(arl + k_first + x);
                    ar[x] = v.x; ar[x + 1] = v.y; ar[x + 2] = v.z; ar[x + 3] = v.w;
                }
                av = fuse_piece<TA>(av, d, ar);
            }
            const uint4* fr = frag + (size_t)t * (NA * kFragsPerTile * 64) + lane;
            if (!BF) {
                uint4 w[NA];
#pragma unroll
                for (int nt = 0; nt < NA; ++nt) w[nt] = fr[nt * 64];
#pragma unroll
                for (int nt = 0; nt < NA; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av.x), __uint_as_float(w[nt].x),
                                                                   acc[nt], 0, 0, 0);
#pragma unroll
                for (int nt = 0; nt < NA; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av.y), __uint_as_float(w[nt].y),
                                                                   acc[nt], 0, 0, 0);
#pragma unroll
                for (int nt = 0; nt < NA; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av.z), __uint_as_float(w[nt].z),
                                                                   acc[nt], 0, 0, 0);
#pragma unroll
                for (int nt = 0; nt < NA; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av.w), __uint_as_float(w[nt].w),
                                                                   acc[nt], 0, 0, 0);
            } else {
                const bf16x8_t ax = __builtin_bit_cast(bf16x8_t, av);
#pragma unroll
                for (int nt = 0; nt < NA; ++nt) {
                    const bf16x8_t bh = __builtin_bit_cast(bf16x8_t, fr[(2 * nt) * 64]);
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax, bh, acc[nt], 0, 0, 0);
                }
#pragma unroll
                for (int nt = 0; nt < NA; ++nt) {
                    const bf16x8_t bl = __builtin_bit_cast(bf16x8_t, fr[(2 * nt + 1) * 64]);
                    acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax, bl, acc[nt], 0, 0, 0);
                }
            }
        };
        for (int t0 = 0; t0 < full; t0 += 2 * PS) {
#pragma unroll
            for (int u = 0; u < PS; ++u) b[u] = load_piece(rowp, t0 + PS + u);
            __builtin_amdgcn_sched_barrier(0);     // the loads stay ahead of the MFMAs
#pragma unroll
            for (int u = 0; u < PS; ++u) multiply(a[u], t0 + u, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < PS; ++u) a[u] = load_piece(rowp, t0 + 2 * PS + u);   // beyond the end: nobody reads it
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < PS; ++u) multiply(b[u], t0 + PS + u, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);
        }
        // the last chunks, fewer than two sets: the first set is loaded already
        if (full + PS < g.chunks) {
#pragma unroll
            for (int u = 0; u < PS; ++u) b[u] = load_piece(rowp, full + PS + u);
        }
#pragma unroll
        for (int u = 0; u < PS; ++u)
            if (full + u < g.chunks) multiply(a[u], full + u, std::true_type{});
#pragma unroll
        for (int u = 0; u < PS; ++u)
            if (full + PS + u < g.chunks) multiply(b[u], full + PS + u, std::true_type{});

        // the next tile's first pieces travel while this one is stored
        const int64_t row0 = tile * 32;
        if (tile + stride < n_tiles) {
            if constexpr (FUSE) {
                rowp = row_ptr_fused(tile + stride, nrk0, nrk1, has);
                load_ds(tile + stride);
                rank_of(tile + 2 * stride, nrk0, nrk1);
            } else {
                rowp = row_ptr(tile + stride);
            }
#pragma unroll
            for (int u = 0; u < PS; ++u) a[u] = load_piece(rowp, u);
        }
        // lane holds column c; register r holds row 8*(r/4) + 4*(lane/32) + r%4
        TC* C = static_cast<TC*>(g.C);
        if (g.stage_off) {
            // A lane's 16 values of a tile are 16 different rows: stored directly they are 2- or
            // 4-byte writes, 128 store instructions per 32 x 256 outputs and more of them than a
            // wavefront may have in flight.  The tile is turned through the wavefront's own
            // 2 or 4 KB of LDS instead and leaves as 16-byte pieces, whole 64- or 128-byte rows.
            constexpr int kPer = 16 / (int)sizeof(TC);        // values per piece
            constexpr int kPieces = 32 / kPer;                // pieces per tile row
            constexpr int kRows = 64 / kPieces;               // tile rows per store instruction
            TC* stg = reinterpret_cast<TC*>(skinny_lds + g.stage_off + wave * (32 * 32 * (int)sizeof(TC)));
            // Scores::kRows: of a row's four lanes lane j keeps the sums of vector j % 2 over the tiles 2k + j / 2
            float sums[(NT + 1) / 2][32 / kRows] = {};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float av1[kPer], av2[kPer];
                if constexpr (SR) {
                    const float* const at = vecs + nt * 32 + lane % kPieces * kPer;
#pragma unroll
                    for (int x = 0; x < kPer; ++x) {
                        av1[x] = at[x];
                        av2[x] = at[NT * 32 + x];
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    stg[(8 * (r / 4) + 4 * gq + (r % 4)) * 32 + c] = from_f32<TC>(acc[nt][r]);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int pass = 0; pass < 32 / kRows; ++pass) {
                    const int row = pass * kRows + lane / kPieces, piece = lane % kPieces;
                    const TC* from = stg + row * 32 + piece * kPer;
                    const int64_t i = row0 + row, n = n0 + nt * 32 + piece * kPer;
                    if constexpr (SR) {
                        float z[kPer], c1 = 0.f, c2 = 0.f;
                        Vec<TC>::unpack(*reinterpret_cast<const uint4*>(from), z);
#pragma unroll
                        for (int x = 0; x < kPer; ++x) {
                            c1 = fmaf(av1[x], z[x], c1);
                            c2 = fmaf(av2[x], z[x], c2);
                        }
                        c1 = quad_sum(c1);
                        c2 = quad_sum(c2);
                        const float own = (lane & 1) ? c2 : c1;
                        sums[nt / 2][pass] = (nt & 1) && (lane & 2) == 0 ? sums[nt / 2][pass] : own;
                        asm volatile("" : "+v"(sums[nt / 2][pass]));     // formed here, not behind the last tile
                    }
                    if (i < g.M) {
                        if (n + kPer <= g.N) {
                            store16(C + i * g.ldc + n, *reinterpret_cast<const uint4*>(from));
                        } else {
                            for (int e = 0; e < kPer && n + e < g.N; ++e) C[i * g.ldc + n + e] = from[e];
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
                if constexpr (SR) __builtin_amdgcn_sched_barrier(0);     // one tile's values of the vectors at a time
            }
            if constexpr (SR) {
                // the slab's heads, [32 rows][heads] of each vector, leave through the staging tile as whole lines
                const int tiles = g.D >> 5, heads = NT / tiles;      // (powers of two, whole heads: scores_with_rows)
                const int lg = 31 - __clz(heads);
                float* const turn = reinterpret_cast<float*>(stg);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                int late = lane;
                asm volatile("" : "+v"(late));     // (addresses formed here, not kept across the products)
                const int vec = late & 1, odd = (late >> 1) & 1;
#pragma unroll
                for (int pass = 0; pass < 32 / kRows; ++pass) {
                    const int row = pass * kRows + late / kPieces;
                    float* const to = turn + ((vec * 32 + row) << lg);
                    if (tiles == 1) {
#pragma unroll
                        for (int k = 0; k < (NT + 1) / 2; ++k)
                            if (2 * k + odd < NT) to[2 * k + odd] = sums[k][pass];
                    } else if constexpr (NT >= 2) {
#pragma unroll
                        for (int k = 0; k < NT / 2; ++k) sums[k][pass] = add_xor2(sums[k][pass]);
                        if (tiles == 2) {
#pragma unroll
                            for (int k = 0; k < NT / 2; ++k)
                                if (!odd) to[k] = sums[k][pass];
                        } else if constexpr (NT >= 4) {
#pragma unroll
                            for (int k = 0; k < NT / 4; ++k)
                                if (!odd) to[k] = sums[2 * k][pass] + sums[2 * k + 1][pass];
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const int h0 = (int)(n0 / g.D);
                for (int x = late; x < 32 << lg; x += 64) {
                    const int64_t i = row0 + (x >> lg);
                    const int h = h0 + (x & (heads - 1));
                    if (i < g.M && h < g.H) {
                        if (g.s1) g.s1[i * g.H + h] = turn[x];
                        if (g.s2) g.s2[i * g.H + h] = turn[(32 << lg) + x];
                    }
                }
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int64_t n = n0 + nt * 32 + c;
                if (n >= g.N) continue;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t i = row0 + 8 * (r / 4) + 4 * gq + (r % 4);
                    if (i < g.M) C[i * g.ldc + n] = from_f32<TC>(acc[nt][r]);
                }
            }
        }
        if (SC && c < 2 * g.H) {
            float* dst = c < g.H ? g.s1 : g.s2;
            const int h = c < g.H ? c : c - g.H;
            if (dst && (h * g.D) / (NT * 32) == (int)blockIdx.y) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t i = row0 + 8 * (r / 4) + 4 * gq + (r % 4);
                    if (i < g.M) dst[i * g.H + h] = acc[NA - 1][r];
                }
            }
        }
    }
}

struct SkinnyPlan {
    int nt = 0;          // accumulator tiles per workgroup slab (1, 2, 4 or 8)
    unsigned slabs = 0;  // column slabs of nt*32
    size_t lds = 0;
    int chunks = 0;
    int stage_off = 0;   // see SkinnyArgs
};

// Whether the skinny kernel applies: the contraction must be at least a 16-byte piece long, and the
// small operand must fit in LDS in at most four column slabs.
bool plan_skinny(int K, int N, int dtype, int extra_tiles, SkinnyPlan* p)
{
    const int elem = dtype == SAR_F32 ? 4 : 2, piece = 16 / elem;
    if (K < piece) return false;
    const int chunk = 2 * piece;
    p->chunks = (K + chunk - 1) / chunk;
    const size_t unit = dtype == SAR_F32 ? 1024 : 2048;
    const int need = (N + 31) / 32;
    int nt = 1;
    while (nt < need && nt < 8) nt *= 2;
    // Outputs go through staging tiles: always for 2-byte
    // outputs (stored directly they are scattered 2-byte writes), for 4-byte outputs when the
    // tiles fit beside the small operand without narrowing the slab
    bool stage = true;
    size_t stage_bytes = (size_t)kSkinnyWaves * 32 * 32 * elem;
    auto fits = [&](int t, size_t extra) {
        return (size_t)p->chunks * (t + extra_tiles) * unit + extra <= kSkinnyMaxLds;
    };
    if (dtype == SAR_F32) {
        while (nt >= 1 && !fits(nt, 0)) nt /= 2;
        if (nt >= 1 && !fits(nt, stage_bytes)) {
            stage = false;
            stage_bytes = 0;
        }
    } else {
        while (nt >= 1 && !fits(nt, stage_bytes)) nt /= 2;
    }
    if (nt < 1) return false;
    p->nt = nt;
    p->slabs = (unsigned)((need + nt - 1) / nt);
    p->lds = (size_t)p->chunks * (nt + extra_tiles) * unit;
    p->stage_off = stage ? (int)p->lds : 0;
    p->lds += stage_bytes;
    return p->slabs <= 4;
}

template <typename TA, typename TC, int NT, Scores SC, bool FUSE, bool RAG>
int launch_skinny_nt(const SkinnyArgs& g, const SkinnyPlan& p, hipStream_t st)
{
    int dev = 0;
    SAR_HIP(hipGetDevice(&dev));
    int n_cu = 0;
    SAR_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    SAR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_skinny<TA, TC, NT, SC, FUSE, RAG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds));
    const int64_t tiles = (g.M + 31) / 32;
    // one workgroup per CU; two where registers (NT <= 4) and LDS leave room
    const int per_cu = (NT <= 4 && 2 * p.lds <= 150 * 1024) ? 2 : 1;
    const int64_t resident = std::max<int64_t>(1, (int64_t)n_cu * per_cu / p.slabs);
    dim3 grid((unsigned)std::max<int64_t>(1, std::min(tiles, resident)), p.slabs, 1);
    k_gemm_skinny<TA, TC, NT, SC, FUSE, RAG><<<grid, kSkinnyThreads, p.lds, st>>>(g);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <typename TA, typename TC, Scores SC = Scores::kNone, bool FUSE = false>
int launch_skinny(const SkinnyArgs& g, const SkinnyPlan& p, hipStream_t st)
{
    auto with = [&](auto ragged) {
        constexpr bool RAG = decltype(ragged)::value;
        switch (p.nt) {
            case 1: return launch_skinny_nt<TA, TC, 1, SC, FUSE, RAG>(g, p, st);
            case 2: return launch_skinny_nt<TA, TC, 2, SC, FUSE, RAG>(g, p, st);
            case 4: return launch_skinny_nt<TA, TC, 4, SC, FUSE, RAG>(g, p, st);
        }
        // (FUSE: not with eight accumulator tiles, see plan_takes_rows_op)
        if constexpr (!FUSE) return launch_skinny_nt<TA, TC, 8, SC, FUSE, RAG>(g, p, st);
        return sar::fail(SAR_ERR_STATE, "rows formed on the fly take at most four accumulator tiles");
    };
    if constexpr (SC != Scores::kTile && !FUSE)
        if (g.K % (16 / (int)sizeof(TA)) != 0) return with(std::true_type{});
    return with(std::false_type{});
}

// Whether a plan can also form the rows of A on the fly (k_gemm_skinny's FUSE): the outputs must
// go through staging tiles, and a tile must hold 32 x H values of ds and 256 of a_r.
bool plan_takes_rows_op(const SkinnyPlan& p, int K, int H, int dtype)
{
    const size_t tile = 32 * 32 * (dtype == SAR_F32 ? 4 : 2);
    // (with eight accumulator tiles the registers are spoken for)
    return p.nt <= 4 && p.stage_off != 0 && K <= 256 && H <= 2 * kDsRegs && (size_t)(32 * H + 256) * 4 <= tile;
}

// Which scores of stored bf16 rows are formed where the rows leave (Scores::kRows): heads of whole staging tiles, a power of
// two of them, that no slab of columns divides (a lane then holds eight values of one head, as a lane of the pass does, and the sums are the
// pass's own), and room for the slab's values of both vectors.  The others are a pass over the stored rows, which costs a read of all of them.  (Bound by
// memory; us, product and pass / together: 3.5 M rows of 128 to 8 x 32 565 + 443 / 696, 313 thousand 71 + 39 / 87, 31 thousand of 256
// to 4 x 64 27 + 19 / 24.)
size_t row_score_bytes(const SkinnyPlan& p) { return (size_t)2 * p.nt * 32 * sizeof(float); }
bool scores_with_rows(int D, const SkinnyPlan& p)
{
    return (D == 32 || D == 64 || D == 128) && p.nt * 32 % D == 0 && p.stage_off != 0 &&
           p.lds + row_score_bytes(p) <= kSkinnyMaxLds;
}

// ---- products whose small operand does not fit in LDS -----------------------
//
// The same two products for the wider layers (400 x 400 fp32 is 640 KB).  A wavefront keeps 32 rows of the
// result, NT tiles of 32 columns wide, in registers and reads its rows of A straight from memory, 16
// bytes per lane, a step of 32 contraction values ahead.  The small operand passes through LDS in the
// same steps, in the order the fragments are consumed (one conflict-free 16-byte read per lane and
// fragment); the next step's values travel while this one is multiplied and are written to the other
// buffer after it, so there is one barrier per step, 64 to 128 matrix instructions of a wavefront.
// The column tiles are dealt evenly to the slabs (400 columns: 7 + 6 tiles), because a 128-wide tiling
// multiplies a quarter for nothing there; the slabs of the same rows are neighbours on one XCD, whose
// L2 serves the rows the second time.
//
// fp32: a lane group holds values 8t+4g .. 8t+4g+3 of a chunk t; swapping the halves of register pairs
//       turns them into the pairs (0,1) (2,3) (4,5) (6,7), so that the contraction runs in its natural order.
// bf16: a chunk is 16 values, hi and lo multiplied in turn (see above).
//
// Bound by the matrix cores in fp32.  Measured before (128 x 128 tiles of both operands staged in LDS,
// widened to fp32 there) and now, forward / dX: 600000 x 400 x 400 fp32 2650 / 2600 -> 1950 / 2010 us (117
// TFLOP/s counting the 14 tiles), bf16 2554 / 1820 -> 787 / 787 us; 5000 x 400 x 400 bf16 54 / 37 -> 17 us.
struct StepArgs {
    const void* A;     // [M, K], row stride lda, contraction index contiguous
    int64_t lda, M;
    const float* B;    // B(k, n) = B[k * sbk + n * sbn]
    int64_t sbk, sbn;
    void* C;           // [M, N], row stride ldc
    int64_t ldc;
    int K, N, slabs;
};

constexpr int kStepWaves = 4;
constexpr int kStepThreads = 64 * kStepWaves;
constexpr int kStepRows = 32 * kStepWaves;
constexpr int kStep = 32;   // contraction values per step

// BK_FAST: the small operand's contiguous direction is the contraction (sbk == 1), otherwise its columns (sbn == 1)
template <typename T, int NT, bool BK_FAST>
__global__ __launch_bounds__(kStepThreads, 2) void k_gemm_steps(StepArgs g)
{
    constexpr bool BF = sizeof(T) == 2;
    constexpr int kChunk = BF ? 16 : 8, kChunks = kStep / kChunk, kVec = 16 / (int)sizeof(T);
    constexpr int kFrags = BF ? 2 : 1;                           // fragments per chunk and tile
    constexpr int kItems = kChunks * NT * (BF ? 64 : 32);        // of 8 values of one column
    constexpr int kPer = (kItems + kStepThreads - 1) / kStepThreads;
    constexpr int kLds = NT * kFrags * 64 + 2;                   // units of a chunk
    __shared__ uint4 frag[2][kChunks * kLds];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, gq = lane >> 5;
    // blocks 8 apart share an XCD: the slabs of one row block
    const int64_t row_block = (int64_t)(blockIdx.x / (8 * g.slabs)) * 8 + blockIdx.x % 8;
    const int n0 = (int)(blockIdx.x / 8 % g.slabs) * NT * 32;
    const int64_t row0 = row_block * kStepRows + wave * 32;
    if (row_block * kStepRows >= g.M) return;
    const T* row = static_cast<const T*>(g.A) + std::min<int64_t>(row0 + c, g.M - 1) * g.lda;
    const int steps = (g.K + kStep - 1) / kStep;

    const int k_last = g.K - kVec, rest = g.K % kVec;
    auto load_a = [&](int step, uint4 (&a)[kChunks]) {
#pragma unroll
        for (int t = 0; t < kChunks; ++t) {
            const int k = step * kStep + t * kChunk + gq * kVec;
            a[t] = load16(row + min(k, k_last));
        }
    };
    // item -> place in LDS, first contraction value in the step, column.  Neighbouring lanes take
    // neighbouring memory: columns, or the four items of a column (128 bytes) where the contraction is
    // the contiguous direction (a line per lane and load there cost a third of the time, 2008 against
    // 2690 us; the two units between chunks keep the four on different banks)
    auto item = [&](int u, int& at, int& kb, int& n) {
        int f, l;
        if (BK_FAST) {
            const int piece = u & 3, col = u >> 2;
            const int t = BF ? piece >> 1 : piece;
            f = t * NT + (col >> 5);
            l = (col & 31) + (BF ? (piece & 1) * 32 : 0);
        } else {
            f = BF ? u >> 6 : u >> 5;
            l = BF ? u & 63 : u & 31;
        }
        const int t = f / NT;
        kb = t * kChunk + (BF ? (l >> 5) * 8 : 0);
        n = n0 + (f % NT) * 32 + (l & 31);
        at = t * kLds + (f % NT) * kFrags * 64 + l;
    };
    // an item's byte offset from the step's first value; the step and the value's place are in the scalar base
    uint32_t from[kPer];
#pragma unroll
    for (int x = 0; x < kPer; ++x) {
        int at, kb, n;
        item(min(tid + x * kStepThreads, kItems - 1), at, kb, n);
        from[x] = (uint32_t)(kb * g.sbk + std::min<int64_t>(n, g.N - 1) * g.sbn) * 4u;
    }
    float bv[kPer][8];
    auto load_b = [&](int step, auto last) {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            if (decltype(last)::value) {
                int at, kb, n;
                item(min(tid + x * kStepThreads, kItems - 1), at, kb, n);
                const float* col = g.B + std::min<int64_t>(n, g.N - 1) * g.sbn;
#pragma unroll
                for (int j = 0; j < 8; ++j) bv[x][j] = col[(int64_t)min(step * kStep + kb + j, g.K - 1) * g.sbk];
            } else if (BK_FAST) {
#pragma unroll
                for (int j = 0; j < 8; j += 4) {
                    const uint4 v = load16(reinterpret_cast<const char*>(g.B + step * kStep + j) + from[x]);
                    bv[x][j] = __uint_as_float(v.x);
                    bv[x][j + 1] = __uint_as_float(v.y);
                    bv[x][j + 2] = __uint_as_float(v.z);
                    bv[x][j + 3] = __uint_as_float(v.w);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    bv[x][j] = *reinterpret_cast<const float*>(
                        reinterpret_cast<const char*>(g.B + (int64_t)(step * kStep + j) * g.sbk) + from[x]);
            }
        }
    };
    // (columns beyond N are another column's values: nothing of them is stored)
    auto store_b = [&](int step, int buf, auto last) {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            const int u = tid + x * kStepThreads;
            if (u >= kItems) break;
            int at, kb, n;
            item(u, at, kb, n);
            kb += step * kStep;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (!decltype(last)::value || kb + j < g.K) ? bv[x][j] : 0.f;
            uint32_t p[4], q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (BF) {
                    const uint32_t h0 = f32_to_bf16_rne(v[2 * j]), h1 = f32_to_bf16_rne(v[2 * j + 1]);
                    p[j] = h0 | (h1 << 16);
                    q[j] = f32_to_bf16_rne(v[2 * j] - __uint_as_float(h0 << 16)) |
                           (f32_to_bf16_rne(v[2 * j + 1] - __uint_as_float(h1 << 16)) << 16);
                } else {
                    p[j] = __float_as_uint(v[2 * j]);          // lane group 0: even values
                    q[j] = __float_as_uint(v[2 * j + 1]);      // lane group 1: odd values
                }
            }
            frag[buf][at] = make_uint4(p[0], p[1], p[2], p[3]);
            frag[buf][at + (BF ? 64 : 32)] = make_uint4(q[0], q[1], q[2], q[3]);
        }
    };

    float16_t acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;

    auto multiply = [&](int buf, int t, const uint4& av) {
        const uint4* fr = frag[buf] + t * kLds + lane;
        if constexpr (BF) {
            const bf16x8_t ax = __builtin_bit_cast(bf16x8_t, av);
            // four tiles at a time, so that no instruction waits for the sums of the one before it
#pragma unroll
            for (int n4 = 0; n4 < NT; n4 += 4) {
                uint4 w[2][4];
#pragma unroll
                for (int nt = n4; nt < NT && nt < n4 + 4; ++nt) {
                    w[0][nt - n4] = fr[(2 * nt) * 64];
                    w[1][nt - n4] = fr[(2 * nt + 1) * 64];
                }
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int nt = n4; nt < NT && nt < n4 + 4; ++nt)
                        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            ax, __builtin_bit_cast(bf16x8_t, w[half][nt - n4]), acc[nt], 0, 0, 0);
            }
        } else {
            // (k0|k4) (k1|k5) -> (k0|k1) (k4|k5), and so for the other two
            const auto lo = __builtin_amdgcn_permlane32_swap(av.x, av.y, false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(av.z, av.w, false, false);
            const float k01 = __uint_as_float(lo[0]), k45 = __uint_as_float(lo[1]);
            const float k23 = __uint_as_float(hi[0]), k67 = __uint_as_float(hi[1]);
#pragma unroll
            for (int n4 = 0; n4 < NT; n4 += 4) {
                uint4 w[4];
#pragma unroll
                for (int nt = n4; nt < NT && nt < n4 + 4; ++nt) w[nt - n4] = fr[nt * 64];
                auto pair = [&](float av2, auto value) {
#pragma unroll
                    for (int nt = n4; nt < NT && nt < n4 + 4; ++nt)
                        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(av2, __uint_as_float(value(w[nt - n4])),
                                                                       acc[nt], 0, 0, 0);
                };
                pair(k01, [](const uint4& v) { return v.x; });
                pair(k23, [](const uint4& v) { return v.y; });
                pair(k45, [](const uint4& v) { return v.z; });
                pair(k67, [](const uint4& v) { return v.w; });
            }
        }
    };

    uint4 a[kChunks], next[kChunks];
    if (g.K < kVec) {
        T v[kVec] = {};
#pragma unroll
        for (int x = 0; x < kVec; ++x)
            if (x < g.K) v[x] = row[x];
#pragma unroll
        for (int t = 0; t < kChunks; ++t) a[t] = __builtin_bit_cast(uint4, v);
    } else {
        load_a(0, a);
    }
    if (steps > 1) {
        load_b(0, std::false_type{});
        store_b(0, 0, std::false_type{});
        __syncthreads();
        for (int step = 0; step + 2 < steps; ++step) {
            load_a(step + 1, next);
            load_b(step + 1, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);     // the loads stay ahead of the MFMAs
#pragma unroll
            for (int t = 0; t < kChunks; ++t) multiply(step & 1, t, a[t]);
            __builtin_amdgcn_sched_barrier(0);
            store_b(step + 1, (step + 1) & 1, std::false_type{});
#pragma unroll
            for (int t = 0; t < kChunks; ++t) a[t] = next[t];
            __syncthreads();
        }
        load_a(steps - 1, next);
        load_b(steps - 1, std::true_type{});
#pragma unroll
        for (int t = 0; t < kChunks; ++t) multiply(steps & 1, t, a[t]);
#pragma unroll
        for (int t = 0; t < kChunks; ++t) a[t] = next[t];
    } else {
        load_b(0, std::true_type{});
    }
    store_b(steps - 1, (steps - 1) & 1, std::true_type{});
    __syncthreads();
    // the last step, where K ends
#pragma unroll
    for (int t = 0; t < kChunks; ++t) {
        const int k0 = (steps - 1) * kStep + t * kChunk, k_first = k0 + gq * kVec;
        if (k0 >= g.K) break;
        uint4 av = a[t];
        if (k_first > k_last && rest != 0 && g.K >= kVec) av = front_of_piece<T>(av, rest);
        const bool beyond = k_first >= g.K;
        av = make_uint4(beyond ? 0u : av.x, beyond ? 0u : av.y, beyond ? 0u : av.z, beyond ? 0u : av.w);
        multiply((steps - 1) & 1, t, av);
    }

    // lane holds column c; register r holds row 8*(r/4) + 4*(lane/32) + r%4
    T* C = static_cast<T*>(g.C);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = n0 + nt * 32 + c;
        if (n >= g.N) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t i = row0 + 8 * (r / 4) + 4 * gq + (r % 4);
            if (i < g.M) C[i * g.ldc + n] = from_f32<T>(acc[nt][r]);
        }
    }
}

// Column tiles per workgroup: at most eight (128 accumulator registers leave two wavefronts per
// SIMD), the slabs as even as they come; with few rows two, so that more workgroups share the work.
template <typename T>
int launch_steps(StepArgs g, hipStream_t st)
{
    const int need = (g.N + 31) / 32;
    const int64_t row_blocks = (g.M + kStepRows - 1) / kStepRows;
    g.slabs = (need + 7) / 8;
    int nt = (need + g.slabs - 1) / g.slabs;
    if (nt <= 4) nt = nt <= 2 ? 2 : 4;
    if (nt > 2 && row_blocks * g.slabs < 256) nt = row_blocks * ((need + 3) / 4) < 256 ? 2 : 4;
    g.slabs = (need + nt - 1) / nt;
    const unsigned grid = (unsigned)((row_blocks + 7) / 8 * 8 * g.slabs);
    auto with = [&](auto bk_fast) {
        constexpr bool BK = decltype(bk_fast)::value;
        switch (nt) {
            case 2: k_gemm_steps<T, 2, BK><<<grid, kStepThreads, 0, st>>>(g); break;
            case 4: k_gemm_steps<T, 4, BK><<<grid, kStepThreads, 0, st>>>(g); break;
            case 5: k_gemm_steps<T, 5, BK><<<grid, kStepThreads, 0, st>>>(g); break;
            case 6: k_gemm_steps<T, 6, BK><<<grid, kStepThreads, 0, st>>>(g); break;
            case 7: k_gemm_steps<T, 7, BK><<<grid, kStepThreads, 0, st>>>(g); break;
            default: k_gemm_steps<T, 8, BK><<<grid, kStepThreads, 0, st>>>(g); break;
        }
    };
    if (g.sbk == 1)
        with(std::true_type{});
    else
        with(std::false_type{});
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// ---- dW = X^T dZ: contraction over the rows ---------------------------------
//
// Here both operands have the contraction index (the node) as their slow
// dimension, the opposite of what an MFMA fragment wants from a lane.  A
// workgroup copies chunks of rows of X (up to 128 columns) and dZ (up to 256
// columns) into LDS as they are (16-byte accesses both sides, double
// buffered, one barrier per chunk) and the wavefronts read their fragments
// column-wise from there: one element per lane and row, which costs LDS
// instructions but no bank conflicts (row strides put the two lane groups of
// a fragment on different banks).  The output tile is 128 x NW, two n-tiles and
// four kf-tiles per wavefront (128 accumulator registers); tiles beyond K or N
// are skipped.  NW = 256: the four wavefronts side by side.  NW = 128: two by
// two, the pairs taking every other row step of a chunk and adding up through
// LDS at the end.  NW = 64: the same with the kf-tiles dealt to the halves of
// a pair.  Rows are split into slabs over the grid; each slab writes its
// partial tile, summed below.  Rows of any width and alignment: the last unit
// of a row that is no whole number of them is read where the row ends and moved
// to its front (RAG).
//
// bf16 rows only: fp32 rows take k_dw_split.  What this measured, before (one 128 x 256 shape, no slab below 128 rows, a
// general tiled kernel for other widths) and now: 254 x 200 over 30000 rows and other widths off 16 bytes 28..59 ->
// 10..25 us.  Two wavefronts per SIMD have to be asked for: with the guarded and the unguarded row step both in it the
// compiler takes one.

constexpr int kDwKf = 128;

constexpr int kDwRows = 32;          // rows per chunk
constexpr int kDwPad = 8;            // LDS row strides: rows 8 apart (the two lane groups) 32 banks apart
constexpr int kDwVec = 8;            // elements per 16 bytes

template <bool FUSE, int NW, bool RAG>
__global__ __launch_bounds__(256, 2) void k_dw(const bf16_t* __restrict__ X, const bf16_t* __restrict__ dZ,
                                            RowsOp op, float* __restrict__ partial, int64_t M, int K, int N,
                                            int64_t rows_per_slab)
{
    using T = bf16_t;
    constexpr int kXUnits = kDwRows * kDwKf / kDwVec / 256;   // 16-byte units per thread and chunk
    constexpr int kDUnits = kDwRows * NW / kDwVec / 256;
    constexpr int kXs = kDwKf + kDwPad, kDs = NW + kDwPad;
    constexpr int kCols = NW / 64, kParts = NW == 256 ? 1 : 2, kKg = 4 / kCols / kParts, kKt = 4 / kKg;
    __shared__ __attribute__((aligned(16))) T Xs[2][kDwRows][kXs];
    __shared__ __attribute__((aligned(16))) T Ds[2][kDwRows][kDs];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, gq = lane >> 5;
    const int kf0 = blockIdx.z * kDwKf, n0 = blockIdx.y * NW;
    const int64_t m_beg = (int64_t)blockIdx.x * rows_per_slab;
    const int64_t m_end = std::min<int64_t>(M, m_beg + rows_per_slab);
    const int cw = wave % kCols, part = (wave / kCols) % kParts, kg = wave / (kCols * kParts);
    // this wavefront's tiles that exist (its kf-tile kt is the workgroup's kt * kKg + kg)
    const int kt_n = min(kKt, ((K - kf0 + 31) / 32 + kKg - 1 - kg) / kKg);
    const int nt_n = max(0, min(2, (N - n0 - 64 * cw + 31) / 32));

    // RAG: the unit in which a row ends is read from the row's last 16 bytes and moved to its front
    // where it is stored (commit); rows shorter than a unit are read value by value
    auto unit = [](const T* row, int col, int width) -> uint4 {
        if constexpr (RAG) {
            if (width < kDwVec) {
                T v[kDwVec] = {};
#pragma unroll
                for (int x = 0; x < kDwVec; ++x)
                    if (x < width) v[x] = row[x];
                return __builtin_bit_cast(uint4, v);
            }
            col = min(col, width - kDwVec);
        }
        return load16(row + col);
    };
    auto placed = [](const uint4& v, int col, int width) -> uint4 {
        if constexpr (RAG) {
            if (width > kDwVec && col < width && col + kDwVec > width) return front_of_piece<T>(v, width % kDwVec);
        }
        return v;
    };
    uint4 gx[kXUnits], gd[kDUnits];
    // FUSE: the rows of dZ are formed here (see RowsOp).  A thread's units keep their column, so its
    // pieces of a_r and its heads are fixed; the row map of a chunk is read one chunk ahead of the
    // rows themselves, which keeps a single level of loads in flight.
    __shared__ __attribute__((aligned(16))) float ars[FUSE ? NW : 4];   // this tile's columns of a_r
    float dsv[FUSE ? kDUnits : 1];
    int hq[FUSE ? kDUnits : 1], rk0[FUSE ? kDUnits : 1], rk1[FUSE ? kDUnits : 1];
    auto fetch_rank = [&](int64_t m0) {
        if constexpr (FUSE) {
#pragma unroll
            for (int q = 0; q < kDUnits; ++q) {
                const int u = tid + 256 * q, row = u / (NW / kDwVec);
                const bool ok = op.rank != nullptr && m0 + row < m_end;
                rk0[q] = ok ? op.rank[m0 + row] : 0;
                rk1[q] = ok ? op.rank[m0 + row + 1] : 0;
            }
        }
    };
    if constexpr (FUSE) {
        // a piece's values four by four: the first four of every piece, then (8-value pieces) the
        // last four, so that neighbouring lanes read neighbouring 16 bytes (no bank conflicts)
        for (int f = tid; f < NW; f += 256) {
            const int piece = f / kDwVec, x = f % kDwVec;
            ars[(x / 4) * (NW / 2) + piece * 4 + (x % 4)] = (op.ds && n0 + f < N) ? op.a_r[n0 + f] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kDUnits; ++q) {
            const int u = tid + 256 * q, col = (u % (NW / kDwVec)) * kDwVec;
            hq[q] = n0 + col < N ? (n0 + col) / op.D : 0;
            dsv[q] = 0.f;
        }
        fetch_rank(m_beg);
        __syncthreads();
    }
    auto fetch = [&](int64_t m0) {
#pragma unroll
        for (int q = 0; q < kXUnits; ++q) {
            const int u = tid + 256 * q, row = u / (kDwKf / kDwVec), col = (u % (kDwKf / kDwVec)) * kDwVec;
            const bool ok = m0 + row < m_end && kf0 + col < K;
            gx[q] = ok ? unit(X + (m0 + row) * K, kf0 + col, K) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int q = 0; q < kDUnits; ++q) {
            const int u = tid + 256 * q, row = u / (NW / kDwVec), col = (u % (NW / kDwVec)) * kDwVec;
            const bool ok = m0 + row < m_end && n0 + col < N;
            if constexpr (FUSE) {
                int64_t from = m0 + row;
                bool has = ok && op.has_E;
                if (op.rank) {
                    from = rk0[q];
                    has = has && rk1[q] > rk0[q];
                }
                gd[q] = has ? *reinterpret_cast<const uint4*>(dZ + from * N + n0 + col) : make_uint4(0u, 0u, 0u, 0u);
                dsv[q] = (ok && op.ds) ? op.ds[(m0 + row) * op.H + hq[q]] : 0.f;
            } else {
                gd[q] = ok ? unit(dZ + (m0 + row) * N, n0 + col, N) : make_uint4(0u, 0u, 0u, 0u);
            }
        }
        fetch_rank(m0 + kDwRows);
    };
    auto commit = [&](int buf) {
#pragma unroll
        for (int q = 0; q < kXUnits; ++q) {
            const int u = tid + 256 * q, row = u / (kDwKf / kDwVec), col = (u % (kDwKf / kDwVec)) * kDwVec;
            *reinterpret_cast<uint4*>(&Xs[buf][row][col]) = placed(gx[q], kf0 + col, K);
        }
#pragma unroll
        for (int q = 0; q < kDUnits; ++q) {
            const int u = tid + 256 * q, row = u / (NW / kDwVec), col = (u % (NW / kDwVec)) * kDwVec;
            if constexpr (FUSE) {
                float arv[kDwVec];
#pragma unroll
                for (int x = 0; x < kDwVec; x += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(ars + (x / 4) * (NW / 2) + (col / kDwVec) * 4);
                    arv[x] = v.x; arv[x + 1] = v.y; arv[x + 2] = v.z; arv[x + 3] = v.w;
                }
                *reinterpret_cast<uint4*>(&Ds[buf][row][col]) = fuse_piece<T>(gd[q], dsv[q], arv);
            } else
                *reinterpret_cast<uint4*>(&Ds[buf][row][col]) = placed(gd[q], n0 + col, N);
        }
    };

    float16_t acc[kKt][2];
#pragma unroll
    for (int a = 0; a < kKt; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

    constexpr int kStep = 16;   // rows per matrix instruction
    // one row step; ALL: every tile of this wavefront exists
    auto step = [&](int buf, int s, auto all) {
        constexpr bool ALL = decltype(all)::value;
        const uint16_t(*xs)[kXs] = reinterpret_cast<const uint16_t(*)[kXs]>(Xs[buf]);
        const uint16_t(*ds)[kDs] = reinterpret_cast<const uint16_t(*)[kDs]>(Ds[buf]);
        const int r0 = kStep * s + 8 * gq;
        auto column = [&](auto tile, int col) -> bf16x8_t {
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = (uint32_t)tile[r0 + 2 * e][col] | ((uint32_t)tile[r0 + 2 * e + 1][col] << 16);
            return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
        };
        bf16x8_t b[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            if (ALL || nt < nt_n) b[nt] = column(ds, 64 * cw + 32 * nt + c);
#pragma unroll
        for (int kt = 0; kt < kKt; ++kt)
            if (ALL || kt < kt_n) {
                const bf16x8_t a = column(xs, 32 * (kt * kKg + kg) + c);
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    if (ALL || nt < nt_n)
                        acc[kt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[nt], acc[kt][nt], 0, 0, 0);
            }
    };
    const bool all = kt_n == kKt && nt_n == 2;

    if (m_beg < m_end) {
        fetch(m_beg);
        commit(0);
    }
    __syncthreads();
    int buf = 0;
    for (int64_t m0 = m_beg; m0 < m_end; m0 += kDwRows, buf ^= 1) {
        const bool more = m0 + kDwRows < m_end;
        if (more) fetch(m0 + kDwRows);
        if (all) {
#pragma unroll
            for (int s = 0; s < kDwRows / kStep / kParts; ++s) step(buf, s * kParts + part, std::true_type{});
        } else {
#pragma unroll
            for (int s = 0; s < kDwRows / kStep / kParts; ++s) step(buf, s * kParts + part, std::false_type{});
        }
        if (more) commit(buf ^ 1);
        __syncthreads();
    }
    if constexpr (kParts == 2) {
        // the second half's sums through LDS, a kf-tile at a time (the operand buffers are free now)
        static_assert(2 * 2 * 16 * 64 * sizeof(float) <= sizeof(Xs), "two wavefronts' kf-tiles");
        float* mine = reinterpret_cast<float*>(&Xs[0][0][0]) + (kg * kCols + cw) * 2 * 16 * 64 + lane;
#pragma unroll
        for (int kt = 0; kt < kKt; ++kt) {
            if (part == 1)
#pragma unroll
                for (int q = 0; q < 32; ++q) mine[q * 64] = acc[kt][q / 16][q % 16];
            __syncthreads();
            if (part == 0)
#pragma unroll
                for (int q = 0; q < 32; ++q) acc[kt][q / 16][q % 16] += mine[q * 64];
            __syncthreads();
        }
        if (part == 1) return;
    }

    // lane holds column c; register r holds row 8*(r/4) + 4*(lane/32) + r%4
    float* out = partial + (int64_t)blockIdx.x * K * N;
#pragma unroll
    for (int kt = 0; kt < kKt; ++kt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int n = n0 + 64 * cw + 32 * nt + c;
            if (n >= N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kf = kf0 + 32 * (kt * kKg + kg) + 8 * (r / 4) + 4 * gq + (r % 4);
                if (kf < K) out[(int64_t)kf * N + n] = acc[kt][nt][r];
            }
        }
}

// dW[k] += sum over slabs of partial[slab][k].  32 consecutive elements per
// workgroup, eight threads per element taking every eighth slab; the eight
// partial sums are added in a fixed order, so the result is reproducible.
// Eight slabs are read at a time: a small dW has few workgroups, and with one
// load in flight per thread they waited 64 times in a row (100 x 36 from 512
// slabs: 18 us).
__global__ __launch_bounds__(256) void k_sum_slabs(const float* __restrict__ partial, int n_slabs, int64_t count,
                                                   float* __restrict__ dW)
{
    __shared__ float part[8][32];
    const int e = threadIdx.x & 31, zl = threadIdx.x >> 5;
    for (int64_t k0 = (int64_t)blockIdx.x * 32; k0 < count; k0 += (int64_t)gridDim.x * 32) {
        const int64_t k = k0 + e;
        float s = 0.f;
        if (k < count)
            for (int z0 = zl; z0 < n_slabs; z0 += 64) {
                float v[8];
#pragma unroll
                for (int x = 0; x < 8; ++x) v[x] = partial[(int64_t)std::min(z0 + 8 * x, n_slabs - 1) * count + k];
#pragma unroll
                for (int x = 0; x < 8; ++x) s = z0 + 8 * x < n_slabs ? s + v[x] : s;
            }
        part[zl][e] = s;
        __syncthreads();
        if (zl == 0 && k < count) {
            float t = part[0][e];
#pragma unroll
            for (int j = 1; j < 8; ++j) t += part[j][e];
            dW[k] += t;
        }
        __syncthreads();
    }
}

// Whether two operands share no memory (the kernels of few rows read an operand again after parts of the result are stored).
bool apart(const void* a, size_t a_bytes, const void* b, size_t b_bytes)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return !a || !b || !a_bytes || !b_bytes || x + a_bytes <= y || y + b_bytes <= x;
}

constexpr int kMaxSlabs = 512;

// How many slabs of rows dW is split into: as many as fill the chip (1024 workgroups), each of at
// least 128 rows.  Where the partial tiles written and read again stay below the operands' own
// bytes, down to 32 rows: a step of few nodes would otherwise wait for a handful of workgroups.
int slabs_for(int64_t n, int K, int F)
{
    const int64_t tiles = (int64_t)((K + 127) / 128) * ((F + 127) / 128);
    const int64_t want = std::min<int64_t>(kMaxSlabs, std::max<int64_t>(1, (1024 + tiles - 1) / tiles));
    const int64_t cheap = std::min(n / 32, n * (K + F) / (2 * (int64_t)K * F));
    return (int)std::max<int64_t>(1, std::min(want, std::max(n / 128, cheap)));
}

}  // namespace

extern "C" int sar_linear_workspace_bytes(int64_t n, int K, int F, size_t* bytes)
{
    SAR_CHECK_ARG(bytes != nullptr, "bytes is null");
    SAR_CHECK_ARG(n >= 0 && K > 0 && F > 0, "need n >= 0, K > 0, F > 0");
    *bytes = (size_t)slabs_for(n, K, F) * K * F * sizeof(float);
    return SAR_OK;
}

extern "C" int sar_linear_fwd(const void* X, const float* W, void* Z, int dtype, int64_t n, int K, int F, int H,
                              int D, const float* a_score, float* score, const float* a_score2, float* score2,
                              void* stream)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    SAR_CHECK_ARG(n >= 0 && K > 0 && F > 0, "need n >= 0, K > 0, F > 0");
    SAR_CHECK_ARG((a_score == nullptr) == (score == nullptr), "a_score and score must be given together");
    SAR_CHECK_ARG((a_score2 == nullptr) == (score2 == nullptr), "a_score2 and score2 must be given together");
    SAR_CHECK_ARG(!(a_score || a_score2) || (H > 0 && D > 0 && H * D == F), "scores need H*D == F");
    if (n == 0) return SAR_OK;
    SAR_CHECK_ARG(X && W && Z, "X, W or Z is null");
    hipStream_t st = sar::as_stream(stream);
    SkinnyPlan plan;
    const bool want_scores = a_score || a_score2;
    // fp32 rows that are no whole number of pieces take the stepwise kernel, whose contraction runs in its
    // natural order, as it always did for them: the scores' signs decide slopes
    const bool rows_whole = dtype == SAR_BF16 || K % 4 == 0;
    // With fp32 rows the scores are two more columns of the product (z_h . a_h = x . (W_h a_h)),
    // equal to the scores of the stored rows up to fp32 rounding.  With bf16 rows they are taken
    // from the STORED (rounded) rows: every later step reads those rows,
    // and a score of the unrounded sums differs from theirs by up to the storage rounding, which
    // is enough to move LeakyReLU's kink for about one edge in a thousand.  (Where the shape allows it they
    // are taken as the rows leave: scores_with_rows.)
    const size_t elem = dtype == SAR_F32 ? 4 : 2;
    const bool alone = apart(X, (size_t)n * K * elem, Z, (size_t)n * F * elem);
    if (want_scores && dtype == SAR_F32 && 2 * H <= 32 && rows_whole && plan_skinny(K, F, dtype, 1, &plan)) {
        if (alone && sar::few_rows(dtype, n, K, F, true, plan.nt))
            return sar::few_fwd(dtype, {X, n, W, Z, K, F, a_score, a_score2, score, score2, H, D}, false, st);
        SkinnyArgs sk{X, K, n, W, F, 1, Z, F, K, F, plan.chunks, a_score, a_score2, score, score2, H, D,
                      plan.stage_off};
        SAR_TRY((launch_skinny<float, float, Scores::kTile>(sk, plan, st)));
        return SAR_OK;
    }
    const bool natural = !(rows_whole && plan_skinny(K, F, dtype, 0, &plan));
    // scores written over X or W, which a caller may be done with, wait until all rows are formed
    auto clear = [&](const float* s) {
        const size_t bytes = (size_t)n * H * sizeof(float);
        return !s || (apart(X, (size_t)n * K * elem, s, bytes) && apart(W, (size_t)K * F * sizeof(float), s, bytes));
    };
    if (alone && sar::few_rows(dtype, n, K, F, false, natural ? 2 : plan.nt)) {
        SAR_TRY(sar::few_fwd(dtype, {X, n, W, Z, K, F, nullptr, nullptr, nullptr, nullptr, 0, 0}, natural, st));
    } else if (!natural) {
        SkinnyArgs sk{X, K, n, W, F, 1, Z, F, K, F, plan.chunks, nullptr, nullptr, nullptr, nullptr, 0, 0,
                      plan.stage_off};
        if (dtype == SAR_F32) {
            SAR_TRY((launch_skinny<float, float>(sk, plan, st)));
        } else if (want_scores && (uintptr_t)Z % 16 == 0 && scores_with_rows(D, plan) && clear(score) && clear(score2)) {
            sk.a1 = a_score;
            sk.a2 = a_score2;
            sk.s1 = score;
            sk.s2 = score2;
            sk.H = H;
            sk.D = D;
            sk.vec_off = (int)plan.lds;
            plan.lds += row_score_bytes(plan);
            SAR_TRY((launch_skinny<bf16_t, bf16_t, Scores::kRows>(sk, plan, st)));
            return SAR_OK;
        } else {
            SAR_TRY((launch_skinny<bf16_t, bf16_t>(sk, plan, st)));
        }
    } else {
        const StepArgs g{X, K, n, W, F, 1, Z, F, K, F, 0};
        SAR_TRY(dtype == SAR_F32 ? launch_steps<float>(g, st) : launch_steps<bf16_t>(g, st));
    }
    // (one pass over the stored rows; with one vector the same vector rides along twice)
    if (a_score || a_score2) {
        const float* a1 = a_score ? a_score : a_score2;
        float* s1 = a_score ? score : score2;
        const float* a2 = a_score2 ? a_score2 : a_score;
        float* s2 = a_score2 ? score2 : score;
        return sar::gat_scores2(Z, dtype, n, H, D, a1, s1, a2, s2, stream);
    }
    return SAR_OK;
}

namespace {

// Whether both products can form the rows `op` describes while they load them (k_dw, k_dw_split,
// k_gemm_skinny and k_dx_split with FUSE): their aligned fast paths, a piece inside one head, the stand-in row
// readable.  dZ here is the stored part E (or the stand-in when there is none).  (k_gemm_skinny's limits bind dX of fp32
// rows too, which k_dx_split forms at any width: what a call without scratch for the rows refuses is as it was.)
bool rows_op_fusable(const void* X, const void* dZ, const RowsOp& op, void* dX, int dtype, int K, int F)
{
    const int elem = dtype == SAR_F32 ? 4 : 2, vec = 16 / elem;
    if (K % vec != 0 || F % vec != 0 || op.D % vec != 0 || op.H * op.D != F || op.H > 2 * kDsRegs) return false;
    if (reinterpret_cast<uintptr_t>(X) % 16 != 0 || reinterpret_cast<uintptr_t>(dZ) % 16 != 0) return false;
    if (op.ds && reinterpret_cast<uintptr_t>(op.a_r) % 16 != 0) return false;
    SkinnyPlan plan;
    if (dX && !(plan_skinny(F, K, dtype, 0, &plan) && plan_takes_rows_op(plan, F, op.H, dtype)))
        return false;
    return true;
}

// The error rows of RowsOp written out (the shapes the two products cannot form on the fly):
// the same fp32 multiply-add and the same rounding as sar_gat_bwd_end's.  A thread's place moves on by the grid's
// length without a division.  PIECES: 16 bytes of a row and head at a time, at any alignment; the last piece of a row
// is moved back to end with it, and its values that the piece before holds are written twice, alike.  Bound by memory:
// 150003 x 47 fp32 26.5 -> 15.0 us against a value at a time, 125001 x 47 bf16 20.0 -> 9.0; 2450000 x 400 fp32 takes
// 1575 (5.0 TB/s).
template <typename T, bool PIECES>
__global__ __launch_bounds__(256) void k_rows_store(const T* E, RowsOp op, T* out, int64_t n, int F)
{
    constexpr int V = PIECES ? 16 / (int)sizeof(T) : 1;
    const int units = (F + V - 1) / V;
    const int64_t step = (int64_t)gridDim.x * 256, first = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t di = step / units;
    const int du = (int)(step - di * units);
    int64_t i = first / units;
    int u = (int)(first - i * units);
    for (; i < n; i += di, u += du) {
        if (u >= units) {
            u -= units;
            if (++i >= n) break;
        }
        const int f = PIECES ? min(u * V, F - V) : u;
        int64_t from = i;
        bool present = op.has_E;
        if (present && op.rank) {
            from = op.rank[i];
            present = op.rank[i + 1] > (int32_t)from;
        }
        const float d = op.ds ? op.ds[i * op.H + (op.H > 1 ? f / op.D : 0)] : 0.f;
        if constexpr (PIECES) {
            uint4 v = present ? load16(E + from * F + f) : make_uint4(0u, 0u, 0u, 0u);
            if (op.ds) {
                float ar[V];
#pragma unroll
                for (int x = 0; x < V; x += 4) {
                    const uint4 p = load16(op.a_r + f + x);
                    ar[x] = __uint_as_float(p.x), ar[x + 1] = __uint_as_float(p.y);
                    ar[x + 2] = __uint_as_float(p.z), ar[x + 3] = __uint_as_float(p.w);
                }
                v = fuse_piece<T>(v, d, ar);
            }
            store16(out + i * F + f, v);
        } else {
            float o = 0.f;
            if (present) {
                if constexpr (sizeof(T) == 2)
                    o = bf16_to_f32(E[from * F + f]);
                else
                    o = E[from * F + f];
            }
            if (op.ds) o = fmaf(d, op.a_r[f], o);
            out[i * F + f] = from_f32<T>(o);
        }
    }
}

int rows_store(const void* E, const RowsOp& op, void* out, int dtype, int64_t n, int F, hipStream_t st)
{
    auto with = [&](auto row) {
        using T = decltype(row);
        // a piece lies within one head
        const int vec = 16 / (int)sizeof(T);
        const bool pieces = F >= vec && (!op.ds || op.H == 1 || op.D % vec == 0);
        const int64_t units = n * (pieces ? (F + vec - 1) / vec : F);
        const unsigned grid = (unsigned)std::min<int64_t>((units + 255) / 256, 16384);
        if (pieces)
            k_rows_store<T, true><<<grid, 256, 0, st>>>(static_cast<const T*>(E), op, static_cast<T*>(out), n, F);
        else
            k_rows_store<T, false><<<grid, 256, 0, st>>>(static_cast<const T*>(E), op, static_cast<T*>(out), n, F);
    };
    if (dtype == SAR_F32)
        with(float{});
    else
        with(bf16_t{});
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// Which fp32 dX goes by pieces (k_dx_split) and which by the fp32 instruction (k_gemm_skinny; stored and formed rows alike).
// Sums of 16 and fewer: not measured.  Up to 32 columns are one tile of the two that k_dx_split takes: 17 to 37% slower (F
// = 100 to 400, 250000 rows 16 columns 28 -> 36, 90 -> 120 us).  Up to 64 columns of rows that end within a line of memory are
// read twice as they stream from memory, in steps of 64 bytes: 1000000 rows F = 100, 200, 400 175 -> 191, 259 -> 319, 476 -> 534
// (whole lines, F = 128, 256: 201 -> 183, 336 -> 315; within reach of the 256 MiB cache, 250000 rows F = 100 47 -> 41).
bool dx_by_split(int64_t n, int K, int F)
{
    if (F <= 16 || K <= 32) return false;
    return !(K <= 64 && F > 64 && F % 32 != 0 && n * F * (int64_t)sizeof(float) > (int64_t)256 << 20);
}

// op == nullptr: dZ is the stored [n,F] operand.  Otherwise dZ is the stored part of the rows
// `op` describes and both products form the rows as they load them.  dZ_rows: its rows, 0 for a stand-in of which no value counts.
int linear_bwd_impl(const void* X, const void* dZ, int64_t dZ_rows, const RowsOp* op, const float* W, float* dW, void* dX, int dtype,
                    int64_t n, int K, int F, void* work, size_t work_bytes, hipStream_t st)
{
    if (!dW && !dX) return SAR_OK;       // (an empty grid is refused by the runtime)
    auto add_slabs = [&](int slabs) -> int {
        const int64_t count = (int64_t)K * F;
        k_sum_slabs<<<(unsigned)std::min<int64_t>((count + 31) / 32, 8192), 256, 0, st>>>(
            static_cast<const float*>(work), slabs, count, dW);
        SAR_LAUNCH_CHECK();
        return SAR_OK;
    };
    const size_t elem = dtype == SAR_F32 ? 4 : 2;
    SkinnyPlan few_plan;
    const bool few_split = dtype == SAR_F32 && dx_by_split(n, K, F);
    const sar::FewBwd few{X, dZ, W, dW, dX, static_cast<float*>(work), n, K, F, slabs_for(n, K, F), few_split,
                          !few_split && !plan_skinny(F, K, dtype, 0, &few_plan)};
    if (sar::few_rows_bwd(dtype, few, op != nullptr) && apart(dX, (size_t)n * K * elem, dZ, (size_t)dZ_rows * F * elem) &&
        (!dW || apart(dX, (size_t)n * K * elem, X, (size_t)n * K * elem))) {
        if (dW) {
            const size_t need = (size_t)slabs_for(n, K, F) * K * F * sizeof(float);
            SAR_CHECK_ARG(work != nullptr && work_bytes >= need, "work_bytes=%zu is below the %zu bytes required",
                          work_bytes, need);
        }
        int slabs = 0;
        SAR_TRY(sar::few_bwd(dtype, few, op, &slabs, st));
        return slabs > 0 ? add_slabs(slabs) : SAR_OK;
    }
    if (dW) {
        int slabs = slabs_for(n, K, F);
        const size_t need = (size_t)slabs_for(n, K, F) * K * F * sizeof(float);
        SAR_CHECK_ARG(work != nullptr && work_bytes >= need, "work_bytes=%zu is below the %zu bytes required",
                      work_bytes, need);
        // dW[K,F] = X^T dZ, contraction over the n rows, split into slabs
        auto slabs_bf16 = [&]() -> int {
            const int64_t rows_per_slab = ((n + slabs - 1) / slabs + kDwRows - 1) / kDwRows * kDwRows;
            auto launch = [&](auto kernel, int nw) {
                const dim3 grid((unsigned)slabs, (unsigned)((F + nw - 1) / nw), (unsigned)((K + kDwKf - 1) / kDwKf));
                kernel<<<grid, 256, 0, st>>>(static_cast<const bf16_t*>(X), static_cast<const bf16_t*>(dZ),
                                             op ? *op : RowsOp{}, static_cast<float*>(work), n, K, F, rows_per_slab);
            };
            auto with = [&](auto fuse, auto ragged) {
                constexpr bool FUSE = decltype(fuse)::value, RAG = decltype(ragged)::value;
                if (F <= 64)
                    launch(k_dw<FUSE, 64, RAG>, 64);
                else if (F <= 128)
                    launch(k_dw<FUSE, 128, RAG>, 128);
                else
                    launch(k_dw<FUSE, 256, RAG>, 256);
            };
            if (op)   // (rows_op_fusable: whole units)
                with(std::true_type{}, std::false_type{});
            else if (K % 8 == 0 && F % 8 == 0)
                with(std::false_type{}, std::false_type{});
            else
                with(std::false_type{}, std::true_type{});
            SAR_LAUNCH_CHECK();
            return SAR_OK;
        };
        if (dtype == SAR_F32)
            SAR_TRY(sar::split_dw(static_cast<const float*>(X), static_cast<const float*>(dZ), op,
                                  static_cast<float*>(work), n, K, F, slabs, &slabs, st));
        else
            SAR_TRY(slabs_bf16());
        SAR_TRY(add_slabs(slabs));
    }
    if (dX) {
        // dX[n,K] = dZ W^T : B(k = f, n = kcol) = W[kcol * F + f]
        SkinnyPlan plan;
        // (dX in the place of dZ: k_dx_split reads a row again after parts of dX are stored, for its other columns and for
        // rows that are redone, k_gemm_skinny of one slab has read its rows by then)
        if (dtype == SAR_F32 && dx_by_split(n, K, F) && dX != dZ) {
            SAR_TRY(sar::split_dx(static_cast<const float*>(dZ), op, W, static_cast<float*>(dX), n, K, F, st));
        } else if (plan_skinny(F, K, dtype, 0, &plan)) {
            SkinnyArgs sk{dZ, F, n, W, 1, F, dX, K, F, K, plan.chunks, nullptr, nullptr, nullptr, nullptr, 0, 0,
                          plan.stage_off};
            if (op) {
                sk.op = *op;
                if (dtype == SAR_F32)
                    SAR_TRY((launch_skinny<float, float, Scores::kNone, true>(sk, plan, st)));
                else
                    SAR_TRY((launch_skinny<bf16_t, bf16_t, Scores::kNone, true>(sk, plan, st)));
            } else if (dtype == SAR_F32) {
                SAR_TRY((launch_skinny<float, float>(sk, plan, st)));
            } else {
                SAR_TRY((launch_skinny<bf16_t, bf16_t>(sk, plan, st)));
            }
        } else {
            if (op) return sar::fail(SAR_ERR_STATE, "rows formed on the fly need the skinny dX kernel");
            const StepArgs g{dZ, F, n, W, 1, F, dX, K, F, K, 0};
            SAR_TRY(dtype == SAR_F32 ? launch_steps<float>(g, st) : launch_steps<bf16_t>(g, st));
        }
    }
    return SAR_OK;
}

}  // namespace

extern "C" int sar_linear_bwd(const void* X, const void* dZ, const float* W, float* dW, void* dX, int dtype,
                              int64_t n, int K, int F, void* work, size_t work_bytes, void* stream)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    SAR_CHECK_ARG(n >= 0 && K > 0 && F > 0, "need n >= 0, K > 0, F > 0");
    if (n == 0) return SAR_OK;
    SAR_CHECK_ARG(dZ != nullptr, "dZ is null");
    SAR_CHECK_ARG(dW == nullptr || X != nullptr, "dW needs X");
    SAR_CHECK_ARG(dX == nullptr || W != nullptr, "dX needs W");
    if (dW) {
        const size_t need = (size_t)slabs_for(n, K, F) * K * F * sizeof(float);
        SAR_CHECK_ARG(work != nullptr && work_bytes >= need, "work_bytes=%zu is below the %zu bytes required",
                      work_bytes, need);
    }
    return linear_bwd_impl(X, dZ, n, nullptr, W, dW, dX, dtype, n, K, F, work, work_bytes, sar::as_stream(stream));
}

extern "C" int sar_linear_bwd_rows(const void* X, const void* E, const int32_t* E_rank, int64_t n_E,
                                   const float* ds, const float* a_r, int H, int D, const float* W, float* dW,
                                   void* dX, int dtype, int64_t n, int K, void* rows, void* work,
                                   size_t work_bytes, void* stream)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    SAR_CHECK_ARG(H > 0 && D > 0, "need H > 0 and D > 0");
    const int F = H * D;
    SAR_CHECK_ARG(n >= 0 && K > 0 && n_E >= 0, "need n >= 0, K > 0, n_E >= 0");
    if (n == 0) return SAR_OK;
    SAR_CHECK_ARG(E != nullptr || E_rank != nullptr || ds != nullptr,
                  "neither stored rows E nor the term ds (x) a_r is given");
    SAR_CHECK_ARG(E != nullptr || n_E == 0, "E is null but n_E = %lld", (long long)n_E);
    SAR_CHECK_ARG(E == nullptr || E_rank != nullptr || n_E == n, "without E_rank, E has one row per node: n_E must be n");
    SAR_CHECK_ARG((ds == nullptr) == (a_r == nullptr), "ds and a_r must be given together");
    SAR_CHECK_ARG(dW == nullptr || X != nullptr, "dW needs X");
    SAR_CHECK_ARG(dX == nullptr || W != nullptr, "dX needs W");
    SAR_CHECK_ARG(rows == nullptr || (rows != E && rows != dX), "rows must not alias E or dX");
    if (dW) {
        const size_t need = (size_t)slabs_for(n, K, F) * K * F * sizeof(float);
        SAR_CHECK_ARG(work != nullptr && work_bytes >= need, "work_bytes=%zu is below the %zu bytes required",
                      work_bytes, need);
    }
    hipStream_t st = sar::as_stream(stream);
    RowsOp op{E_rank, ds, a_r, H, D, (E != nullptr && n_E > 0) ? 1 : 0};
    if (!op.has_E && !ds) {
        // no stored row and no rank-one term: E_p = 0, dW gets nothing and dX is zero
        if (dX) SAR_TRY(rows_store(nullptr, RowsOp{}, dX, dtype, n, K, st));
        return SAR_OK;
    }
    // where no row is stored the kernels still need an address they may read a row from
    const void* stored = op.has_E ? E : static_cast<const void*>(a_r ? a_r : ds);
    if (!rows && rows_op_fusable(X, stored, op, dX, dtype, K, F))
        return linear_bwd_impl(X, stored, op.has_E ? n_E : 0, &op, W, dW, dX, dtype, n, K, F, work, work_bytes, st);
    if (!rows)
        return sar::fail(SAR_ERR_UNSUPPORTED,
                         "this shape (K=%d, H=%d, D=%d) cannot form the error rows inside the products: pass `rows`, "
                         "[n,F] values of scratch, and they are written out first", K, H, D);
    SAR_TRY(rows_store(E, op, rows, dtype, n, F, st));
    return linear_bwd_impl(X, rows, n, nullptr, W, dW, dX, dtype, n, K, F, work, work_bytes, st);
}
