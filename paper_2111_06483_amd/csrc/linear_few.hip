// The dense transform of few rows.
//
// The kernels of linear.hip and linear_split.hip lay the small operand out in LDS for workgroups that walk over many rows.
// Where there are only a few hundred or thousand rows that layout is most of the time: 462 rows 256 x 256 with scores
// took 40 us, of which the products of a wavefront are 17 (five tiles one after the other on 30 of 256 CUs) and the
// staging the rest; now 19, of which the score columns are more than half (8.8 without).  Here a wavefront has one tile of
// 32 x 32 results and reads both operands' fragments straight from memory, several chunks ahead, without LDS or a barrier: as
// many wavefronts as there are tiles, each a chain of a few microseconds.  The second reader of a row or column finds it in
// L1 or L2.  The two backward products of a call are one launch.
//
// Z and dX are the same sums in the same order as in the kernels named beside each function, bit for bit; dW has the same terms in
// an order of its own.
#include <algorithm>
#include <type_traits>

#include "linear_few.h"
#include "linear_pieces.h"
#include "sar_internal.h"

namespace {

using namespace sar;

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;

__device__ inline uint4 zero_if(bool zero, const uint4& v)
{
    return make_uint4(zero ? 0u : v.x, zero ? 0u : v.y, zero ? 0u : v.z, zero ? 0u : v.w);
}

// ---- C = A B by the fp32 instruction, or bf16 rows (k_gemm_skinny; NAT: k_gemm_steps) ----
//
// ALONG: B's contiguous direction is the contraction (dX).  TAIL: K is no whole number of chunks.  FUSE: the rows of A are
// formed (RowsOp).
template <typename T, bool ALONG, bool NAT, bool FUSE, bool TAIL>
struct Product {
    static constexpr bool BF = sizeof(T) == 2;
    static constexpr int kVec = 16 / (int)sizeof(T), kChunk = 2 * kVec;
    static constexpr int kAhead = BF ? 4 : 8;          // chunks on their way
    static_assert(!FUSE || (ALONG && !NAT), "formed rows are those of dX");

    struct Slot {
        uint4 a;
        float b[kVec];
        float ar[FUSE ? kVec : 1], ds;
    };

    const FewArgs& g;
    const RowsOp& op;
    int lane, c, gq, chunks, n0, k_last;
    int64_t row0;
    const T* row;
    const float* col;
    const float* ds_row;
    float inv_D;
    bool has = true;

    __device__ inline Product(const FewArgs& g_, const RowsOp& op_, int64_t tile, int n0_)
        : g(g_), op(op_), n0(n0_), row0(tile * 32)
    {
        lane = threadIdx.x & 63, c = lane & 31, gq = lane >> 5;
        chunks = (g.K + kChunk - 1) / kChunk;
        k_last = g.K - kVec;
        const int64_t i = std::min<int64_t>(row0 + c, g.M - 1);
        int64_t from = i;
        if constexpr (FUSE) {
            inv_D = 1.f / (float)op.D;
            ds_row = op.ds ? op.ds + i * op.H : nullptr;
            has = op.has_E;
            if (has && op.rank) {
                from = op.rank[i];
                has = op.rank[i + 1] > (int32_t)from;
            }
            if (!has) from = 0;                        // (a readable stand-in)
        }
        row = static_cast<const T*>(g.A) + from * g.K;
        const int n = min(n0 + c, g.N - 1);
        col = ALONG ? g.B + (int64_t)n * g.K : g.B + n;
    }

    // contraction value of a lane's B fragment j of chunk t, without ALONG
    __device__ inline int k_of(int t, int j) const { return NAT && !BF ? t * kChunk + 2 * j + gq : t * kChunk + gq * kVec + j; }

    __device__ inline void load_a(int t, Slot& s) const
    {
        const int k = t * kChunk + gq * kVec;
        s.a = load16(row + (TAIL ? min(k, k_last) : k));
        if constexpr (FUSE) {
            if (op.ds) {
                const int ka = TAIL ? min(k, k_last) : k;
                s.ds = ds_row[min((int)(((float)ka + 0.5f) * inv_D), op.H - 1)];
#pragma unroll
                for (int x = 0; x < kVec; x += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(op.a_r + ka + x);
                    s.ar[x] = v.x, s.ar[x + 1] = v.y, s.ar[x + 2] = v.z, s.ar[x + 3] = v.w;
                }
            }
        }
    }
    __device__ inline void load(int t, Slot& s) const
    {
        load_a(t, s);
        if constexpr (ALONG) {
#pragma unroll
            for (int x = 0; x < kVec; x += 4) {
                const int k = t * kChunk + gq * kVec + x;
                const uint4 v = load16(col + (TAIL ? min(k, g.K - 4) : k));
                s.b[x] = __uint_as_float(v.x), s.b[x + 1] = __uint_as_float(v.y);
                s.b[x + 2] = __uint_as_float(v.z), s.b[x + 3] = __uint_as_float(v.w);
            }
        } else if constexpr (TAIL) {
#pragma unroll
            for (int j = 0; j < kVec; ++j) s.b[j] = col[min(k_of(t, j), g.K - 1) * g.N];
        } else {
            // (the chunk's place is in the scalar base)
            const int lane_off = (NAT && !BF ? gq : gq * kVec) * g.N;
#pragma unroll
            for (int j = 0; j < kVec; ++j) s.b[j] = (col + (t * kChunk + (NAT && !BF ? 2 * j : j)) * g.N)[lane_off];
        }
    }
    __device__ inline uint4 value_a(int t, const Slot& s) const
    {
        uint4 a = s.a;
        const int k = t * kChunk + gq * kVec;
        if constexpr (TAIL) {
            const int rest = g.K % kVec;
            if (rest != 0 && k > k_last) a = front_of_piece<T>(a, rest);
        }
        if constexpr (FUSE) {
            a = zero_if(!has, a);
            if (op.ds) a = fuse_piece<T>(a, s.ds, s.ar);
        }
        if constexpr (TAIL) a = zero_if(k >= g.K, a);
        return a;
    }
    __device__ inline void value_b(int t, const Slot& s, float (&b)[kVec]) const
    {
        if constexpr (!TAIL) {
#pragma unroll
            for (int j = 0; j < kVec; ++j) b[j] = s.b[j];
        } else if constexpr (ALONG) {
#pragma unroll
            for (int x = 0; x < kVec; x += 4) {
                const int k = t * kChunk + gq * kVec + x;
                uint4 v = make_uint4(__float_as_uint(s.b[x]), __float_as_uint(s.b[x + 1]), __float_as_uint(s.b[x + 2]),
                                     __float_as_uint(s.b[x + 3]));
                if (g.K % 4 != 0 && k > g.K - 4) v = front_of_piece<float>(v, g.K % 4);
                v = zero_if(k >= g.K, v);
                b[x] = __uint_as_float(v.x), b[x + 1] = __uint_as_float(v.y);
                b[x + 2] = __uint_as_float(v.z), b[x + 3] = __uint_as_float(v.w);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kVec; ++j) b[j] = k_of(t, j) < g.K ? s.b[j] : 0.f;
        }
    }
    static __device__ inline void multiply(const uint4& a, const float (&b)[kVec], float16_t& acc)
    {
        if constexpr (BF) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t h0 = f32_to_bf16_rne(b[2 * j]), h1 = f32_to_bf16_rne(b[2 * j + 1]);
                hi[j] = h0 | (h1 << 16);
                lo[j] = f32_to_bf16_rne(b[2 * j] - __uint_as_float(h0 << 16)) |
                        (f32_to_bf16_rne(b[2 * j + 1] - __uint_as_float(h1 << 16)) << 16);
            }
            const bf16x8_t ax = __builtin_bit_cast(bf16x8_t, a);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                ax, __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3])), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                ax, __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3])), acc, 0, 0, 0);
        } else if constexpr (NAT) {
            // (k0|k4) (k1|k5) -> (k0|k1) (k4|k5), and so for the other two
            const auto p = __builtin_amdgcn_permlane32_swap(a.x, a.y, false, false);
            const auto q = __builtin_amdgcn_permlane32_swap(a.z, a.w, false, false);
            float w[4] = {b[0], b[1], b[2], b[3]};
            if constexpr (ALONG) {
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(b[0]), __float_as_uint(b[1]), false, false);
                const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(b[2]), __float_as_uint(b[3]), false, false);
                w[0] = __uint_as_float(r[0]), w[1] = __uint_as_float(s[0]);
                w[2] = __uint_as_float(r[1]), w[3] = __uint_as_float(s[1]);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(p[0]), w[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(q[0]), w[1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(p[1]), w[2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(q[1]), w[3], acc, 0, 0, 0);
        } else {
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), b[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), b[1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), b[2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), b[3], acc, 0, 0, 0);
        }
    }
    // the contraction: get(t, slot) starts chunk t's loads, use(t, slot) multiplies it
    template <typename Get, typename Use>
    __device__ inline void contract(Get get, Use use) const
    {
        Slot s[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) get(min(u, chunks - 1), s[u]);
        const int full = chunks / kAhead * kAhead;
#pragma unroll 1
        for (int t = 0; t < full; t += kAhead) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                use(t + u, s[u]);
                get(min(t + kAhead + u, chunks - 1), s[u]);      // (beyond the end: nobody reads it)
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead - 1; ++u)
            if (full + u < chunks) use(full + u, s[u]);
    }
    __device__ inline float16_t sums() const
    {
        float16_t acc = {};
        contract([&](int t, Slot& s) SAR_INLINE { load(t, s); },
                 [&](int t, const Slot& s) SAR_INLINE {
                     float b[kVec];
                     value_b(t, s, b);
                     multiply(value_a(t, s), b, acc);
                 });
        return acc;
    }
    // lane holds column c; register r holds row 8 (r/4) + 4 (lane/32) + r%4
    __device__ inline void store(const float16_t& acc) const
    {
        const int n = n0 + c;
        if (n >= g.N) return;
        T* to = static_cast<T*>(g.C) + n;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t i = row0 + 8 * (r / 4) + 4 * gq + (r % 4);
            if (i < g.M) to[i * g.N] = from_f32<T>(acc[r]);
        }
    }
};

// The score columns of four row tiles: W_h a_h of every contraction value first, by all eight wavefronts, as k_gemm_skinny
// forms it (a head's products one after the other), in LDS as the fragments of one column tile.  Rows of W pass through LDS
// score_rows() at a time, the next ones on their way meanwhile.
constexpr int kScoreWaves = 8;

__host__ __device__ inline int score_pitch(int N) { return (N + 3) / 4 * 4 + 4; }
// (16 K values: eight 16-byte loads a thread)
__host__ __device__ inline int score_rows(int K, int N)
{
    const int most = N <= 64 ? 256 : N <= 128 ? 128 : 64;
    return K < most ? (K + 63) / 64 * 64 : most;
}

template <bool TAIL>
__device__ inline void score_columns(const FewArgs& g, int64_t tile, bool live, float* lds)
{
    using P = Product<float, false, false, false, TAIL>;
    constexpr int kThreads = 64 * kScoreWaves, kPer = 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quads = (g.N + 3) / 4, pitch = score_pitch(g.N), cols = 2 * g.H, most = score_rows(g.K, g.N);
    const bool whole = g.D % 4 == 0, even = g.N % 4 == 0;
    const int chunks = (g.K + 7) / 8;
    float* frag = lds;                                  // [chunks][64 lanes][4]
    float* as = frag + chunks * 256;                    // [2][pitch]
    float* rows = as + 2 * pitch;                       // [most][pitch]
    uint4 v[kPer];
    // units of four values x0 + u * kThreads of the rows from k0 on (behind their end: the last one again)
    auto fetch = [&](int k0, int x0) SAR_INLINE {
        const int last = min(most, g.K - k0) * quads - 1;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int x = min(x0 + u * kThreads, last), k = x / quads, f = min(4 * (x - k * quads), g.N - 4);
            v[u] = load16(g.B + (k0 + k) * g.N + f);
        }
    };
    auto keep = [&](int k0, int x0) SAR_INLINE {
        const int last = min(most, g.K - k0) * quads - 1;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int x = min(x0 + u * kThreads, last), k = x / quads, f = min(4 * (x - k * quads), g.N - 4);
            float* to = rows + k * pitch + f;
            if (even) {
                *reinterpret_cast<uint4*>(to) = v[u];
            } else {
                to[0] = __uint_as_float(v[u].x), to[1] = __uint_as_float(v[u].y);
                to[2] = __uint_as_float(v[u].z), to[3] = __uint_as_float(v[u].w);
            }
        }
    };
    fetch(0, tid);
    for (int x = tid; x < chunks * 64; x += kThreads) reinterpret_cast<float4*>(frag)[x] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int x = tid; x < g.N; x += kThreads) {
        as[x] = g.a1 ? g.a1[x] : 0.f;
        as[pitch + x] = g.a2 ? g.a2[x] : 0.f;
    }
    for (int k0 = 0; k0 < g.K; k0 += most) {
        const int n_rows = min(most, g.K - k0);
        if (k0) __syncthreads();
        keep(k0, tid);
        for (int x0 = tid + kPer * kThreads; x0 < n_rows * quads; x0 += kPer * kThreads) {
            fetch(k0, x0);
            keep(k0, x0);
        }
        __syncthreads();
        if (k0 + most < g.K) fetch(k0 + most, tid);
        // a wavefront takes one column of 64 rows at a time
        const int blocks = (n_rows + 63) / 64;
        for (int task = wave; task < blocks * cols; task += kScoreWaves) {
            const int col = task / blocks, kk = task % blocks * 64 + lane, k = k0 + kk;
            if (kk >= n_rows) continue;
            const int h = col < g.H ? col : col - g.H;
            const float* a = as + (col < g.H ? 0 : pitch) + h * g.D;
            const float* w = rows + kk * pitch + h * g.D;
            float sum = 0.f;
            if (whole) {
#pragma unroll 8
                for (int d = 0; d < g.D; d += 4) {
                    const float4 w4 = *reinterpret_cast<const float4*>(w + d), a4 = *reinterpret_cast<const float4*>(a + d);
                    sum = fmaf(w4.x, a4.x, sum);
                    sum = fmaf(w4.y, a4.y, sum);
                    sum = fmaf(w4.z, a4.z, sum);
                    sum = fmaf(w4.w, a4.w, sum);
                }
            } else {
#pragma unroll 8
                for (int d = 0; d < g.D; ++d) sum = fmaf(w[d], a[d], sum);
            }
            frag[(k / 8 * 64 + (k / 4 % 2) * 32 + col) * 4 + k % 4] = sum;
        }
    }
    __syncthreads();
    if (!live) return;
    RowsOp none{};
    const P p(g, none, tile, 0);
    float16_t acc = {};
    p.contract([&](int t, typename P::Slot& s) SAR_INLINE { p.load_a(t, s); },
               [&](int t, const typename P::Slot& s) SAR_INLINE {
                   const float4 w = *reinterpret_cast<const float4*>(frag + (t * 64 + p.lane) * 4);
                   const float b[4] = {w.x, w.y, w.z, w.w};
                   P::multiply(p.value_a(t, s), b, acc);
               });
    if (p.c >= cols) return;
    float* dst = p.c < g.H ? g.s1 : g.s2;
    const int h = p.c < g.H ? p.c : p.c - g.H;
    if (!dst) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t i = p.row0 + 8 * (r / 4) + 4 * p.gq + (r % 4);
        if (i < g.M) dst[i * g.H + h] = acc[r];
    }
}

size_t score_lds(int K, int N)
{
    return ((size_t)(K + 7) / 8 * 256 + (size_t)(score_rows(K, N) + 2) * score_pitch(N)) * sizeof(float);
}

constexpr int fwd_waves(bool scores) { return scores ? kScoreWaves : kWaves; }

template <typename T, bool NAT, bool TAIL, bool SC>
__global__ __launch_bounds__(64 * fwd_waves(SC)) void k_few_fwd(FewArgs g)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = (int64_t)blockIdx.x * kWaves + wave;
    const bool live = wave < kWaves && tile * 32 < g.M;
    if constexpr (SC) {
        extern __shared__ __attribute__((aligned(16))) float few_lds[];
        // (the longest workgroups first)
        if (blockIdx.y == 0) return score_columns<TAIL>(g, tile, live, few_lds);
    }
    if (!live) return;
    RowsOp none{};
    const Product<T, false, NAT, false, TAIL> p(g, none, tile, ((int)blockIdx.y - (SC ? 1 : 0)) * 32);
    p.store(p.sums());
}

// ---- dX = dZ W^T of fp32 rows by three bf16 pieces per value (k_dx_split) ----
template <bool FUSE>
__device__ inline void dx_split_tile(const FewArgs& g, const RowsOp& op, int64_t tile, int n0)
{
    constexpr int kStep = 16, kAhead = FUSE ? 3 : 4;
    const int lane = threadIdx.x & 63, c = lane & 31, gq = lane >> 5;
    const int64_t row0 = tile * 32, i = std::min<int64_t>(row0 + c, g.M - 1);
    const int steps = (g.K + kStep - 1) / kStep, k_last = g.K - 4, rest = g.K % 4;
    const float inv_D = FUSE ? 1.f / (float)op.D : 0.f;
    bool has = true;
    int64_t from = i;
    if constexpr (FUSE) {
        has = op.has_E;
        if (has && op.rank) {
            from = op.rank[i];
            has = op.rank[i + 1] > (int32_t)from;
        }
        if (!has) from = 0;
    }
    const float* row = static_cast<const float*>(g.A) + from * g.K;
    const float* ds_row = FUSE && op.ds ? op.ds + i * op.H : nullptr;
    const float* col = g.B + (int64_t)min(n0 + c, g.N - 1) * g.K;
    struct Slot {
        uint4 a[2], b[2], ar[FUSE ? 2 : 1];
        float ds[FUSE ? 2 : 1];
    };
    auto load = [&](int step, Slot& s) SAR_INLINE {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = min(step * kStep + gq * 8 + 4 * p, k_last);
            s.a[p] = load16(row + k);
            s.b[p] = load16(col + k);
            if constexpr (FUSE) {
                if (op.ds) {
                    s.ds[p] = ds_row[min((int)(((float)k + 0.5f) * inv_D), op.H - 1)];
                    s.ar[p] = load16(op.a_r + k);
                }
            }
        }
    };
    uint32_t low = ~0u;
    auto values = [&](int step, const Slot& s, uint32_t turned, float (&x)[8], float (&w)[8]) SAR_INLINE {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = step * kStep + gq * 8 + 4 * p;
            uint4 a = s.a[p], b = s.b[p];
            if (step == steps - 1 && k > k_last) {
                if (rest != 0) a = front_of_piece<float>(a, rest), b = front_of_piece<float>(b, rest);
                a = zero_if(k >= g.K, a), b = zero_if(k >= g.K, b);
            }
            if constexpr (FUSE) {
                a = zero_if(!has, a);
                if (op.ds) {
                    const float r4[4] = {__uint_as_float(s.ar[p].x), __uint_as_float(s.ar[p].y), __uint_as_float(s.ar[p].z),
                                         __uint_as_float(s.ar[p].w)};
                    a = zero_if(k >= g.K, fuse_piece<float>(a, s.ds[p], r4));
                }
            }
            low = lowest(lowest(low, a), b);
            const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[4 * p + j] = __uint_as_float(av[j] ^ turned);
                w[4 * p + j] = __uint_as_float(bv[j]);
            }
        }
    };
    float16_t acc = {};
    Slot s[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(min(u, steps - 1), s[u]);
    auto use = [&](int step, const Slot& slot) SAR_INLINE {
        float x[8], w[8];
        values(step, slot, (uint32_t)(c + step) << 31, x, w);
        uint4 xp[3], wp[3];
        split8(x, xp);
        split8(w, wp);
        float16_t sum;
        multiply_split(xp, wp, sum);
        const float sign = step % 2 ? -1.f : 1.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = fmaf(r % 2 ? -sign : sign, sum[r], acc[r]);
    };
    const int full = steps / kAhead * kAhead;
#pragma unroll 1
    for (int t = 0; t < full; t += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            use(t + u, s[u]);
            load(min(t + kAhead + u, steps - 1), s[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < kAhead - 1; ++u)
        if (full + u < steps) use(full + u, s[u]);

    if (__any(low < kLowBits || not_finite(acc))) {
        acc = float16_t{};
#pragma unroll 1
        for (int t = 0; t < steps; ++t) {
            float x[8], w[8];
            load(t, s[0]);
            values(t, s[0], 0, x, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], w[j], acc, 0, 0, 0);
        }
    }
    const int n = n0 + c;
    if (n >= g.N) return;
    float* to = static_cast<float*>(g.C) + n;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t at = row0 + 8 * (r / 4) + 4 * gq + (r % 4);
        if (at < g.M) to[at * g.N] = acc[r];
    }
}

// ---- dW = X^T dZ (k_dw_split, k_dw) ----
//
// The four wavefronts of a workgroup take groups of 32 rows of a slab in turn and add their tiles of 32 x 32 up through LDS,
// in order.  Sums of 32 rows are added up eight at a time, and these sums one after the other: one running sum over all rows of a
// wavefront, up to 2048 where many columns leave few slabs, is further off 64 bits than the sums of many rows, whose slabs are short
// (normal operands, bf16 32768 x 64, F = 1024 2.8e-7 of the result against 1.28e-7, and 1.02e-7 by eights; fp32 20480 rows of it
// 1.37e-7, 1.08e-7 and 1.0e-7).  The time is the same.
// A lane reads its column of both operands, a group ahead.  FUSE: the row map of a group is read two groups
// ahead, one entry a lane.
struct DwArgs {
    const void* X;
    const void* dZ;
    float* out;        // partial sums [slabs][K][F], or (slabs == 1) dW itself, added to
    int64_t n;
    int groups;        // of 32 rows, in a slab
    int K, F, slabs;
};
constexpr int kGroup = 32;

template <typename T, bool FUSE>
__device__ inline void dw_tile(const DwArgs& g, const RowsOp& op, int slab, int kf0, int n0, int wave,
                               float (&part)[kWaves - 1][16][64])
{
    constexpr bool BF = sizeof(T) == 2;
    using Raw = std::conditional_t<BF, uint16_t, float>;
    const int lane = threadIdx.x & 63, c = lane & 31, gq = lane >> 5, n_rows = (int)g.n;
    const int m_end = min(n_rows, (slab + 1) * g.groups * kGroup);
    const int m_first = (slab * g.groups + wave) * kGroup;
    constexpr int kTurn = kWaves * kGroup, kRun = 8;
    const int xc = min(kf0 + c, g.K - 1), dc = min(n0 + c, g.F - 1);
    const Raw* X = static_cast<const Raw*>(g.X);
    const Raw* D = static_cast<const Raw*>(g.dZ);
    // (no rank-one term: any readable value times zero)
    const bool with_ds = FUSE && op.ds != nullptr;
    const float* ds = with_ds ? op.ds + dc / op.D : static_cast<const float*>(g.dZ);
    const int ds_ld = with_ds ? op.H : 0;
    const float ar = with_ds ? op.a_r[dc] : 0.f;
    struct Slot {
        Raw x[16], d[16];
        float ds[FUSE ? 16 : 1];
        uint32_t absent;       // FUSE: a bit for each of the lane's rows that E does not have
    };
    int map = 0;
    auto fetch_map = [&](int m0) SAR_INLINE {
        if constexpr (FUSE) {
            if (op.rank) map = op.rank[min(m0 + min(lane, 32), n_rows)];
        }
    };
    // (rows behind the end: the last row's values, zeroed when they are used)
    auto load = [&](int m0, Slot& s) SAR_INLINE {
        uint32_t row[16], from[16];
        if (m0 + kGroup <= n_rows) {
#pragma unroll
            for (int r = 0; r < 16; ++r) row[r] = m0 + 8 * gq + 16 * (r / 8) + r % 8;
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) row[r] = min(m0 + 8 * gq + 16 * (r / 8) + r % 8, n_rows - 1);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) from[r] = row[r];
        if constexpr (FUSE) {
            s.absent = 0u;
            if (!op.has_E) {
                s.absent = ~0u;
#pragma unroll
                for (int r = 0; r < 16; ++r) from[r] = 0;
            } else if (op.rank) {
#pragma unroll
                for (int r = 0; r < 16; r += 8) {
                    int at[9];
#pragma unroll
                    for (int j = 0; j < 9; ++j) at[j] = __shfl(map, 2 * r + 8 * gq + j);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const bool has = at[j + 1] > at[j];
                        s.absent |= has ? 0u : 1u << (r + j);
                        from[r + j] = has ? at[j] : 0;
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s.x[r] = X[row[r] * (uint32_t)g.K + xc];
            s.d[r] = D[from[r] * (uint32_t)g.F + dc];
            if constexpr (FUSE) s.ds[r] = ds[row[r] * (uint32_t)ds_ld];
        }
        fetch_map(m0 + kTurn);
    };
    uint32_t low = ~0u;
    float16_t acc, run;
    // one group of 32 rows, added to run; keep: by the fp32 instruction
    auto use = [&](int m0, const Slot& s, auto keep) SAR_INLINE {
        constexpr bool KEEP = decltype(keep)::value;
        const float sign = m0 & 32 ? -1.f : 1.f;
        float xv[2][8], dv[2][8];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if constexpr (BF) {
                xv[r / 8][r % 8] = __uint_as_float((uint32_t)s.x[r] << 16);
                dv[r / 8][r % 8] = __uint_as_float((uint32_t)s.d[r] << 16);
            } else {
                xv[r / 8][r % 8] = s.x[r];
                dv[r / 8][r % 8] = s.d[r];
            }
            if constexpr (FUSE) {
                float& d = dv[r / 8][r % 8];
                d = s.absent >> r & 1 ? 0.f : d;
                d = fmaf(with_ds ? s.ds[r] : 0.f, ar, d);
            }
        }
        if (m0 + kGroup > m_end) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = m0 + 8 * gq + 16 * (r / 8) + r % 8 < m_end;
                xv[r / 8][r % 8] = in ? xv[r / 8][r % 8] : 0.f;
                dv[r / 8][r % 8] = in ? dv[r / 8][r % 8] : 0.f;
            }
        }
        if constexpr (BF) {
            float16_t sum = {};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const auto packed = [](const float (&v)[8]) {
                    return __builtin_bit_cast(bf16x8_t, make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]),
                                                                   pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7])));
                };
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(packed(xv[t]), packed(dv[t]), sum, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) run[r] += sum[r];
        } else {
            float16_t sum = {};
            if constexpr (!KEEP) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    low = min(low, min(2u * __float_as_uint(xv[r / 8][r % 8]) - 1u, 2u * __float_as_uint(dv[r / 8][r % 8]) - 1u));
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) xv[r / 8][r % 8] *= sign;
            if constexpr (KEEP) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        sum = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[t][j], dv[t][j], sum, 0, 0, 0);
            } else {
                uint4 ap[2][3], bp[2][3];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    split8(xv[t], ap[t]);
                    split8(dv[t], bp[t]);
                }
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ap[h][kTerm[t][0]]),
                                                                      __builtin_bit_cast(bf16x8_t, bp[h][kTerm[t][1]]), sum,
                                                                      0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) run[r] = fmaf(sign, sum[r], run[r]);
        }
    };
    auto rows = [&](auto keep) SAR_INLINE {
        acc = float16_t{};
        run = float16_t{};
        if (m_first >= m_end) return;
        Slot s[2];
        fetch_map(m_first);
        load(m_first, s[0]);
#pragma unroll 1
        for (int m0 = m_first; m0 < m_end; m0 += 2 * kTurn) {
            load(m0 + kTurn, s[1]);
            use(m0, s[0], keep);
            if (m0 + kTurn >= m_end) break;
            load(m0 + 2 * kTurn, s[0]);
            use(m0 + kTurn, s[1], keep);
            if ((m0 - m_first) % (kRun * kTurn) == (kRun - 2) * kTurn) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += run[r], run[r] = 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += run[r];
    };
    if constexpr (BF) {
        rows(std::false_type{});
    } else {
        // (sums of one or two products are closer by the fp32 instruction)
        if (g.n > 2) rows(std::false_type{});
        if (g.n <= 2 || __any(low < kLowBits || not_finite(acc))) rows(std::true_type{});
    }
    if (wave > 0)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[wave - 1][r][lane] = acc[r];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += part[w][r][lane];
    const int n = n0 + c;
    if (n >= g.F) return;
    float* out = g.out + (int64_t)slab * g.K * g.F + n;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int kf = kf0 + 8 * (r / 4) + 4 * gq + (r % 4);
        if (kf < g.K) out[(int64_t)kf * g.F] = g.slabs == 1 ? out[(int64_t)kf * g.F] + acc[r] : acc[r];
    }
}

// The workgroups of dX (x_groups times its column tiles, or none), whose chains are the longer ones, then those of dW.
template <typename T, bool SPLIT, bool NAT, bool FUSE, bool TAIL>
__global__ __launch_bounds__(kThreads, 2) void k_few_bwd(FewArgs g, DwArgs w, RowsOp op, int dx_blocks, int x_groups)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = (int)blockIdx.x;
    if (b >= dx_blocks) {
        __shared__ float part[kWaves - 1][16][64];
        const int n_tiles = (w.F + 31) / 32, k_tiles = (w.K + 31) / 32, id = b - dx_blocks;
        return dw_tile<T, FUSE>(w, op, id / (n_tiles * k_tiles), id / n_tiles % k_tiles * 32, id % n_tiles * 32, wave, part);
    }
    const int64_t tile = (int64_t)(b % x_groups) * kWaves + wave;
    if (tile * 32 >= g.M) return;
    const int n0 = b / x_groups * 32;
    if constexpr (SPLIT) {
        dx_split_tile<FUSE>(g, op, tile, n0);
    } else {
        const Product<T, true, NAT, FUSE, TAIL> p(g, op, tile, n0);
        p.store(p.sums());
    }
}

template <typename T>
int launch_fwd(const FewArgs& g, bool natural, hipStream_t st)
{
    constexpr int kChunk = 32 / (int)sizeof(T);
    const bool scores = g.s1 || g.s2, tail = g.K % kChunk != 0;
    // (four tiles a workgroup in either case: eight would share the SIMDs of one CU beside idle ones)
    const dim3 grid((unsigned)((g.M + 32 * kWaves - 1) / (32 * kWaves)), (unsigned)((g.N + 31) / 32 + (scores ? 1 : 0)));
    auto with = [&](auto nat, auto tl, auto sc) -> int {
        constexpr bool NAT = decltype(nat)::value, TAIL = decltype(tl)::value, SC = decltype(sc)::value;
        if constexpr (!SC || (sizeof(T) == 4 && !NAT)) {
            auto fn = k_few_fwd<T, NAT, TAIL, SC>;
            const size_t lds = SC ? score_lds(g.K, g.N) : 0;
            if (SC)
                SAR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)lds));
            fn<<<grid, 64 * fwd_waves(SC), lds, st>>>(g);
            SAR_LAUNCH_CHECK();
            return SAR_OK;
        } else {
            return fail(SAR_ERR_STATE, "scores beside the product are those of fp32 rows of whole pieces");
        }
    };
    auto with_tail = [&](auto nat, auto sc) {
        return tail ? with(nat, std::true_type{}, sc) : with(nat, std::false_type{}, sc);
    };
    if constexpr (sizeof(T) == 4)
        if (natural) return with_tail(std::true_type{}, std::false_type{});
    return scores ? with_tail(std::false_type{}, std::true_type{}) : with_tail(std::false_type{}, std::false_type{});
}

template <typename T>
int launch_bwd(const FewArgs& g, const DwArgs& w, const FewBwd& b, const RowsOp* op, hipStream_t st)
{
    constexpr int kChunk = 32 / (int)sizeof(T);
    const int dw_blocks = b.dW ? w.slabs * ((w.F + 31) / 32) * ((w.K + 31) / 32) : 0;
    const int x_groups = (int)((g.M + 32 * kWaves - 1) / (32 * kWaves));
    const int dx_blocks = b.dX ? x_groups * ((g.N + 31) / 32) : 0;
    const unsigned grid = (unsigned)(dx_blocks + dw_blocks);
    const RowsOp o = op ? *op : RowsOp{};
    auto go = [&](auto kernel) -> int {
        kernel<<<grid, kThreads, 0, st>>>(g, w, o, dx_blocks, x_groups);
        SAR_LAUNCH_CHECK();
        return SAR_OK;
    };
    const bool tail = g.K % kChunk != 0;
    if constexpr (sizeof(T) == 4) {
        if (b.split) return op ? go(k_few_bwd<T, true, false, true, false>) : go(k_few_bwd<T, true, false, false, false>);
        if (b.natural && !op)
            return tail ? go(k_few_bwd<T, false, true, false, true>) : go(k_few_bwd<T, false, true, false, false>);
    }
    if (op) return tail ? go(k_few_bwd<T, false, false, true, true>) : go(k_few_bwd<T, false, false, true, false>);
    return tail ? go(k_few_bwd<T, false, false, false, true>) : go(k_few_bwd<T, false, false, false, false>);
}

}  // namespace

namespace sar {

// Offsets within an operand are 32-bit numbers here.
static bool small_operands(int64_t n, int K, int F)
{
    return n * std::max(K, F) < (1 << 30) && (int64_t)K * F < (1 << 28);
}

// Workgroups of four tiles of 32 x 32: 256 of them are one wavefront per SIMD.
static int64_t workgroups(int64_t n, int N) { return (n + 32 * kWaves - 1) / (32 * kWaves) * ((N + 31) / 32); }

// The lines are drawn by workgroups.  The other kernel's wavefronts form `wide` tiles one after the other, so it takes the longer
// the more these are while the chip has room for all of them side by side; with more tiles than that, reading both operands
// from memory for each costs more than staging one of them.  us, the other kernel / this one: fp32 with scores, 64 -> 64 (wide 2)
// 2000 rows 10.1 / 7.4, 20000 17.8 / 9.2; 256 -> 64 (2) 10000 rows 26.0 / 14.5, 20000 26.6 / 24.5; 256 -> 256 (4) 100 rows
// 39.5 / 18.8, 5000 41.7 / 20.4, 10000 41.9 / 39.7, 20000 59.8 / 67.2; 100 -> 256 (8) 5000 32.1 / 11.8, 10000 32.7 / 21.3, 20000
// 34.0 / 37.3.  Without: 256 -> 256 500 23.8 / 8.8, 5000 24.8 / 17.8, 10000 25.4 / 27.4; 128 -> 256 (8) 10000 26.3 / 18.0, 20000
// 27.4 / 27.5.  bf16: 256 -> 256 (4) 500 12.7 / 6.1, 5000 13.7 / 9.8, 10000 14.0 / 15.5; 256 -> 64 (2) 10000 7.8 / 6.4, 20000 8.2 /
// 9.9.  By workgroups and not tiles: a few beyond 256 wait for a round of their own (512 -> 400, bf16 2432 rows 13.6 / 10.0, 2496
// rows 13.9 / 16.0).  A long contraction is one chain here, and where the other kernel has few tiles as well that one's loads
// are the wider: 1024 -> 128 and fewer, fp32 27 / 29, bf16 12 / 16.5 (-> 256: 22.5 / 16.3); bf16 of one column tile 512 -> 16
// 7.7 / 9.9, 256 -> 16 6.4 / 7.1 and, from 8000 rows on, 9.4 / 7.2 (32 -> 16: 4.6 / 4.1 from the fewest on).
bool few_rows(int dtype, int64_t n, int K, int N, bool scores, int wide)
{
    const bool f32 = dtype == SAR_F32;
    if (K < (f32 ? 4 : 8) || !small_operands(n, K, N)) return false;
    if (scores && (N < 4 || score_lds(K, N) > 160 * 1024)) return false;
    const int64_t w = workgroups(n, N);
    if (K > 512 && N <= 128) return false;
    if (!f32 && N <= 32 && K > 64 && (w < 64 || K > 256)) return false;
    return w <= (scores ? 80 * (wide + 1) : 128 * wide);
}

int few_fwd(int dtype, const FewArgs& g, bool natural, hipStream_t st)
{
    return dtype == SAR_F32 ? launch_fwd<float>(g, natural, st) : launch_fwd<bf16_t>(g, natural, st);
}

// Partial sums of dW, and the groups of rows of one.
struct DwPlan {
    int slabs, groups;
    int chain() const { return (groups + kWaves - 1) / kWaves; }      // of a wavefront
};
static DwPlan plan_dw(int64_t n, int K, int F, bool dX, int most_slabs)
{
    const int64_t tiles = (int64_t)((K + 31) / 32) * ((F + 31) / 32), groups = (n + kGroup - 1) / kGroup;
    // (two groups a wavefront are sooner done than a launch that adds slabs up; beside dX, half of the chip)
    const int64_t want = groups <= 2 * kWaves ? 1 : std::max<int64_t>(1, (dX ? 256 : 512) / tiles);
    const int64_t s = std::min<int64_t>({want, (int64_t)most_slabs, (groups + kWaves - 1) / kWaves});
    const int64_t per = (groups + s - 1) / s;
    return {(int)((groups + per - 1) / per), (int)per};
}

// us, the kernels for many rows / this one.  Both products, with the slabs' sum (dX by its workgroups as above, dW of as many
// rows beside it): fp32, formed rows, 64 -> 64 200 rows 18.8 / 8.8, 5000 20.1 / 9.2; 256 -> 256 600 41.0 / 17.8, 2500 43.5 / 23.3,
// 5000 45.9 / 43.3; 128 -> 256 2500 41.8 / 20.2, 10000 46.7 / 45.0; stored rows, 256 -> 256 2500 38.2 / 19.0, 10000 49.3 / 49.1.
// bf16, formed rows, 256 -> 256 600 42.9 / 15.3, 5000 47.7 / 32.3, 10000 51.5 / 55.9; 128 -> 256 10000 48.1 / 33.7; stored, 100 ->
// 256 2500 40.2 / 13.1, 10000 43.9 / 22.4.  (dX before dW in the grid and dW on half of the chip: 1300 rows 256 -> 256 24.5 -> 18.6.)
// From 512 columns of dZ on beyond one wavefront per SIMD two share it on long chains: bf16 128 -> 2048 16384 rows 91 / 165, 8192 52 /
// 44; fp32 100 -> 512 10240 52 / 60.
// dX alone: the other kernel has the chip to itself too.  fp32 64 -> 128 20480 rows 11.4 / 14.4, 15360 10.9 / 8.6; bf16 512 ->
// 256 4096 23.8 / 17.1, 64 -> 256 32768 14.3 / 17.5, 16384 13.1 / 9.7; where that kernel passes W through LDS in steps (natural) it
// has as many wavefronts: 1024 -> 256 2048 rows 10.4 / 17.1, 1024 9.7 / 9.7, 512 -> 512 2432 13.8 / 26.3, 1400 13.9 / 14.7.  Chains
// of more than 512 values only where they fill the SIMDs: 64 -> 1024 16384 26.0 / 25.8, 3200 21.1 / 25.2, 64 -> 2048 52.8 / 46.2,
// 39.7 / 45.9.  One column tile: the other kernel has no tiles to go through one after the other.  fp32 32 -> 128 10240 rows 10.7 /
// 8.6, 4096 7.7 / 8.6; bf16 16384 8.9 / 7.0, 65536 10.8 / 11.5, 6500 6.1 / 7.0; 32 -> 512 16384 12.9 / 15.2; formed rows cost that
// one a staging of ds for every row (fp32 32 -> 256 4096 14.2 / 12.5, bf16 65536 20.6 / 19.5).
// dW alone by the groups of 32 rows that a wavefront sums up: eight cost as much as there (fp32 64 -> 512 15360 rows 21.0 / 22.2, 100
// -> 1024 10240, twenty, 33 / 48; bf16 64 -> 512 16384 19 / 15, 32 -> 512 49152, twelve, 22.2 / 26.3, 256 -> 1024 2848, twelve,
// 27 / 19).
bool few_rows_bwd(int dtype, const FewBwd& b, bool formed)
{
    const bool f32 = dtype == SAR_F32;
    const int K = b.K, F = b.F;
    if (F < (f32 ? 4 : 8) || !small_operands(b.n, K, F)) return false;
    const int64_t w = workgroups(b.n, K), one = 256, most = f32 ? 320 : 512;
    if (b.dX && b.dW) return w <= (F <= (f32 ? 256 : 400) ? most : one);
    if (b.dW) return w <= most && plan_dw(b.n, K, F, false, b.most_slabs).chain() <= (!f32 && K > 64 ? 12 : 8);
    if (K <= 32 && F > 32) {
        if (formed) return w <= most;
        if (F > 1024) return w <= one && (f32 || K <= 16);
        return w >= 64 && w <= (F < 64 && !f32 ? most : one) && (f32 || F <= 400);
    }
    if (f32) return w <= (F <= 32 ? most : one);
    if (F <= 128) return w <= most;
    if (F <= 400) return w <= (K > 64 && !b.natural ? most : one);
    return w <= one && !b.natural && (F <= 512 || w > 192);
}

int few_bwd(int dtype, const FewBwd& b, const RowsOp* op, int* slabs, hipStream_t st)
{
    const FewArgs g{b.dZ, b.n, b.W, b.dX, b.F, b.K, nullptr, nullptr, nullptr, nullptr, 0, 0};
    DwArgs w{b.X, b.dZ, b.work, b.n, 0, b.K, b.F, 0};
    *slabs = 0;
    if (b.dW) {
        const DwPlan p = plan_dw(b.n, b.K, b.F, b.dX != nullptr, b.most_slabs);
        w.groups = p.groups;
        w.slabs = p.slabs;
        if (w.slabs == 1)
            w.out = b.dW;
        else
            *slabs = w.slabs;
    }
    return dtype == SAR_F32 ? launch_bwd<float>(g, w, b, op, st) : launch_bwd<bf16_t>(g, w, b, op, st);
}

}  // namespace sar
