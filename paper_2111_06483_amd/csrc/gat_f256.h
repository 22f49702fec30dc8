// Fused attention kernels specialised for rows of F = 256 values (1 KiB fp32 or
// 512 B bf16): the whole wavefront covers one row, lane x owns features
// 4x..4x+3, and a head is a group of LPH = D/4 consecutive lanes.
//
// Per-edge scalars (score, softmax weight, score gradient) are not computed
// redundantly by every lane of a head.  Edges are taken in sub-batches of up
// to B, and inside a head group lane k works on edge k of the sub-batch: the
// scores of B edges x H heads are formed by one instruction stream, then each
// weight is broadcast back to its head group (DS_SWIZZLE) for the
// multiply-add with the gathered row.  Row addresses come from scalar
// registers (V_READLANE of the coalesced index chunk), so the gathers are
// SGPR-base + lane-offset loads with up to B rows in flight per wavefront.
//
// Two lane geometries.  Exact: the row is 256 contiguous values, lane x owns
// 4x..4x+3.  Padded (template flag PAD): the launch covers 64/LPH heads of any
// width D <= 4*LPH (D a multiple of 4) inside rows of stride `ld`; head h sits in
// lanes [h*LPH, (h+1)*LPH), lane k of it owns features h*D + 4k.. while 4k < D
// and is idle otherwise (it still takes its turn at the per-edge scalars).  That
// brings head widths such as 100 and rows wider than one wavefront (several
// launches over groups of heads) onto these kernels.  Layers whose heads leave
// half of the lanes or more, and head widths that are no multiple of 4, have
// kernels of their own (gat_slots.h).
#pragma once

#include <type_traits>

#include "../../include/sar_mi355x.h"
#include "gather_common.h"
#include "sar_internal.h"

namespace sar {
namespace f256 {

constexpr int kF = 256;

// ---- cross-lane helpers (wave64, DPP rows of 16 lanes) --------------------

template <int CTRL>
__device__ inline float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ inline int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
constexpr int kRowShr = 0x110;         // + n: lane r of a row of 16 reads lane r - n (0 where there is none)
constexpr int kRowShl = 0x100;         // + n: lane r reads lane r + n
constexpr int kQuadXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141;  // lane r of 8 reads lane 7 - r
constexpr int kRowMirror = 0x140;      // lane r of 16 reads lane 15 - r
constexpr int kRowRor8 = 0x128;
constexpr int kQuadReverse = 0x1B;     // quad_perm [3,2,1,0]
constexpr int kRowNewBcast = 0x150;    // + n: every lane of a row of 16 reads the row's lane n

// Of each 32 lanes, the value of the lane at this one's place in the lower row of 16, and in the upper row; and the same of
// the lower and upper 32.  (v_permlane16_swap, v_permlane32_swap of a value with itself: vector instructions, where
// ds_swizzle and ds_bpermute queue up for the LDS crossbar and are waited for.)
struct Pair {
    float lo, hi;
};
__device__ inline Pair rows_of_32(float v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ inline Pair halves_of_64(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}

struct OpSum {
    static __device__ inline float f(float a, float b) { return a + b; }
};
struct OpMax {
    static __device__ inline float f(float a, float b) { return fmaxf(a, b); }
};

// All-reduce over each group of LPH consecutive lanes (LPH = 1..64, power of two).  Every step pairs lanes
// that read each other (a mirror image counts as lane ^ 4, lane ^ 8: the quads, and then the eights, hold
// one value each by then), so every lane of the group ends with the SAME BITS, those of the sum by lane ^ 1,
// lane ^ 2, lane ^ 4 ...  Rotations by 4 and 8 lanes would take as many instructions, but each quad would
// add the four quads in an order of its own: lanes that store the same value, and the edges that different
// lanes speak for, would differ in last bits.
template <int LPH, typename Op>
__device__ inline float group_all(float v)
{
    if constexpr (LPH >= 2) v = Op::f(v, dpp<kQuadXor1>(v));
    if constexpr (LPH >= 4) v = Op::f(v, dpp<kQuadXor2>(v));
    if constexpr (LPH >= 8) v = Op::f(v, dpp<kRowHalfMirror>(v));
    if constexpr (LPH >= 16) v = Op::f(v, dpp<kRowMirror>(v));
    if constexpr (LPH >= 32) {
        const Pair p = rows_of_32(v);
        v = Op::f(p.lo, p.hi);
    }
    if constexpr (LPH >= 64) {
        const Pair p = halves_of_64(v);
        v = Op::f(p.lo, p.hi);
    }
    return v;
}

// A value of every lane of a head group, made ready to be handed to the whole group lane by lane: of<K>() is lane K's (K < 16).
// DPP: one vector instruction each (a scalar where the group is the wavefront), after three for groups of 8 lanes and one
// for 32.  Otherwise ds_swizzle, which leaves the vector units alone: measured (us, ds_swizzle / DPP), 8 lanes by head slices 25 M
// edges forward 2283 / 2249, by rows 201 M edges of bf16 9610 / 9730; 16 lanes 1.5 M edges of bf16, a long row deciding, 276 /
// 282; 32 lanes 122 M edges of 4 x 100 backward 36400 / 35700.
template <int LPH, bool DPP = LPH == 4 || LPH == 32>
struct Spread {
    int lo, hi;
    __device__ inline explicit Spread(int v) : lo(v), hi(v)
    {
        if constexpr (DPP && LPH == 8) {     // lo: the lower quad's values in both quads, hi: the upper quad's
            const int m = dpp_i<kRowHalfMirror>(v);
            lo = __builtin_amdgcn_update_dpp(v, m, kQuadReverse, 0xf, 0xa, false);
            hi = __builtin_amdgcn_update_dpp(v, m, kQuadReverse, 0xf, 0x5, false);
        } else if constexpr (DPP && LPH == 32) {
            lo = __float_as_int(rows_of_32(__int_as_float(v)).lo);
        }
    }
    __device__ inline explicit Spread(uint32_t v) : Spread((int)v) {}
    __device__ inline explicit Spread(float v) : Spread(__float_as_int(v)) {}
    template <int K>
    __device__ inline int of_int() const
    {
        static_assert(K < LPH && K < 16, "a lane of the group's first row");
        if constexpr (LPH == 64)
            return __builtin_amdgcn_readlane(lo, K);
        else if constexpr (!DPP)
            return __builtin_amdgcn_ds_swizzle(lo, K << 5 | (0x1f & ~(LPH - 1)));
        else if constexpr (LPH <= 8)
            return __builtin_amdgcn_mov_dpp(K < 4 ? lo : hi, K % 4 * 0x55, 0xf, 0xf, true);     // quad_perm [K,K,K,K]
        else
            return __builtin_amdgcn_mov_dpp(lo, kRowNewBcast + K, 0xf, 0xf, true);
    }
    template <int K>
    __device__ inline float of() const
    {
        return __int_as_float(of_int<K>());
    }
};

// Sums of 8 per-lane values over each group of LPH consecutive lanes, one sum per lane: the lane
// at position k of its group (k % 8 for LPH > 8) returns the group's sum of c[k % 8].  Eight
// separate all-reductions would move every value through every step; here the lanes first split
// the eight values between them while they add (pairs, quads, eights: 4 + 2 + 1 exchanges), and
// only one value per lane takes the remaining log2(LPH / 8) steps.
// Measured: a gain from LPH = 32 on, where each all-reduction takes steps through the LDS crossbar
// (bf16 4 x 128 and 2 x 256: 3 to 10% per pass); within 16 lanes the eight independent DPP chains
// of the separate all-reductions are as fast or faster.
constexpr int kScatterSumsFrom = 32;
template <int LPH>
__device__ inline float group_sums8(const float (&c)[8])
{
    static_assert(LPH >= 8, "eight lanes share eight sums");
    const int k = threadIdx.x;           // groups start at multiples of 8: the low bits are the position
    const bool b0 = k & 1, b1 = k & 2, b2 = k & 4;
    float v1[4], v2[2];
#pragma unroll
    for (int m = 0; m < 4; ++m) {        // the partner (lane ^ 1) takes the values of the other parity
        const float mine = b0 ? c[2 * m + 1] : c[2 * m], send = b0 ? c[2 * m] : c[2 * m + 1];
        v1[m] = mine + dpp<kQuadXor1>(send);
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {        // lane ^ 2
        const float mine = b1 ? v1[2 * n + 1] : v1[2 * n], send = b1 ? v1[2 * n] : v1[2 * n + 1];
        v2[n] = mine + dpp<kQuadXor2>(send);
    }
    const float mine = b2 ? v2[1] : v2[0], send = b2 ? v2[0] : v2[1];
    // lane ^ 4 = the mirror image within 8 lanes (lane ^ 7) of the quad's reverse (lane ^ 3)
    float v = mine + dpp<kQuadReverse>(dpp<kRowHalfMirror>(send));
    if constexpr (LPH >= 16) v += dpp<kRowRor8>(v);
    if constexpr (LPH >= 32) {
        const Pair p = rows_of_32(v);
        v = p.lo + p.hi;
    }
    if constexpr (LPH >= 64) {
        const Pair p = halves_of_64(v);
        v = p.lo + p.hi;
    }
    return v;
}

template <int N, typename Fn>
__device__ inline void static_for(Fn&& fn)
{
    if constexpr (N > 0) {
        static_for<N - 1>(fn);
        fn(std::integral_constant<int, N - 1>{});
    }
}

// ---- row access: 4 values per lane ---------------------------------------

template <typename T>
struct Row4;
template <>
struct Row4<float> {
    using Raw = float4;
    static __device__ inline Raw load(const float* row, int lane) { return reinterpret_cast<const float4*>(row)[lane]; }
    static __device__ inline void unpack(const Raw& r, float (&v)[4])
    {
        v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
    }
    static __device__ inline void store(float* row, int lane, const float (&v)[4])
    {
        reinterpret_cast<float4*>(row)[lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
};
template <>
struct Row4<bf16_t> {
    using Raw = uint2;
    static __device__ inline Raw load(const bf16_t* row, int lane) { return reinterpret_cast<const uint2*>(row)[lane]; }
    static __device__ inline void unpack(const Raw& r, float (&v)[4])
    {
        v[0] = __uint_as_float(r.x << 16);
        v[1] = __uint_as_float(r.x & 0xffff0000u);
        v[2] = __uint_as_float(r.y << 16);
        v[3] = __uint_as_float(r.y & 0xffff0000u);
    }
    static __device__ inline void store(bf16_t* row, int lane, const float (&v)[4])
    {
        uint2 r;
        r.x = pack2_bf16(v[0], v[1]);
        r.y = pack2_bf16(v[2], v[3]);
        reinterpret_cast<uint2*>(row)[lane] = r;
    }
};

// Accesses of 4 values at any value's alignment (gfx950 takes unaligned vector accesses).
struct __attribute__((packed, aligned(4))) F32x4Any {
    float x, y, z, w;
};
struct __attribute__((packed, aligned(2))) Bf16x4Any {
    uint32_t x, y;
};
template <typename T, bool ANY>
__device__ inline typename Row4<T>::Raw load_raw(const T* p)
{
    if constexpr (!ANY) {
        return *reinterpret_cast<const typename Row4<T>::Raw*>(p);
    } else if constexpr (sizeof(T) == 4) {
        const F32x4Any r = *reinterpret_cast<const F32x4Any*>(p);
        return make_float4(r.x, r.y, r.z, r.w);
    } else {
        const Bf16x4Any r = *reinterpret_cast<const Bf16x4Any*>(p);
        return make_uint2(r.x, r.y);
    }
}
template <typename T, bool ANY>
__device__ inline void store4(T* p, const float (&v)[4])
{
    if constexpr (!ANY)
        Row4<T>::store(p, 0, v);
    else if constexpr (sizeof(T) == 4)
        *reinterpret_cast<F32x4Any*>(p) = F32x4Any{v[0], v[1], v[2], v[3]};
    else
        *reinterpret_cast<Bf16x4Any*>(p) = Bf16x4Any{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
}

// The lane's 4 values of a row (zeros for an idle lane of the padded geometry).
template <typename T, bool PAD>
__device__ inline typename Row4<T>::Raw load_lane(const T* row, int foff, bool on)
{
    using Raw = typename Row4<T>::Raw;
    if constexpr (PAD) {
        Raw r{};
        if (on) r = *reinterpret_cast<const Raw*>(row + foff);
        return r;
    } else {
        return *reinterpret_cast<const Raw*>(row + foff);
    }
}
template <typename T, bool PAD>
__device__ inline void store_lane(T* row, int foff, bool on, const float (&v)[4])
{
    if (!PAD || on) Row4<T>::store(row + foff, 0, v);
}

// The 64 bits of lane `from` (uniform).
__device__ inline uint64_t readlane64(uint64_t v, int from)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, from);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), from);
    return (uint64_t)hi << 32 | lo;
}

struct Tabs {
    const void* Z[SAR_MAX_BLOCKS];
    const float* t[SAR_MAX_BLOCKS];
};

__device__ inline float leaky2(float u, float slope) { return u > 0.f ? u : slope * u; }

// t_j in log2 units, rounded before it meets s_i in the backward kernels (never one multiply-add with the sum
// that follows): the sum's sign chooses the slope, and it has to come out alike in every kernel.  A score of
// exactly zero, s_i = -t_j, then is one here as well.
__device__ inline float score_log2(float t)
{
#pragma clang fp contract(off)
    return t * kLog2e;
}

// ------------------------------------------------------------------ forward

struct FwdP {
    const int32_t* indptr;
    const uint32_t* indices;
    const uint32_t* rows;
    int64_t n_rows, n_long;
    int64_t n_hub;       // workgroups of more than four wavefronts: the rows that all of them share
    const void* Z;
    const float* t;      // source score halves, or null with FLY (formed from a_l and the gathered row)
    const float* a_l;
    const float* s;
    float* m;
    float* l;
    float* acc;
    void* out;
    float* L;
    int H;
    int tag_shift;
    float slope;
    int act;             // SAR_ACT_*: applied to the normalised output rows (ALL only)
    int ld, ldh, D;      // padded geometry: row stride (values), stride of the per-head arrays, head width
};

template <int LPH>
struct FwdState {
    float m2;       // running maximum (log2 units), uniform inside a head group
    float l;        // this lane's share of the running denominator
    float acc[4];   // running numerator for the lane's 4 features
};

// One 64-edge chunk position `mine`(lane) holds; folds edges [0,cnt) of it.  Over all blocks the lanes look up the addresses of
// their edges' rows, all at once, and a batch takes them from there: looked up edge by edge in the launch's table, every row's
// load waited for a scalar load of its own.
template <typename T, int LPH, int B, bool ALL, bool FLY, bool PAD>
__device__ inline void fwd_chunk(FwdState<LPH>& st, const FwdP& a, const GlobalPtr<const void>* s_Z,
                                 const GlobalPtr<const float>* s_t, uint32_t mine, int cnt, int foff, bool on, int h, int k,
                                 float s2, const float (&al)[4])
{
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    uint64_t row = 0;
    if constexpr (ALL) row = s_Z[mine >> a.tag_shift].bits + (uint64_t)(mine & mask) * (uint32_t)(ld * (int)sizeof(T));
    // Shipped scores: lane k of every head group reads its edge's, a batch ahead, so that the weights are ready when
    // the rows arrive (8 heads of 32 bf16 values, 9 M edges: the kernel 1231 -> 1169 us).
    auto shipped = [&](int k0) {
        const uint32_t my = (uint32_t)__shfl((int)mine, min(k0 + min(k, B - 1), cnt - 1));
        const float* tb = ALL ? s_t[my >> a.tag_shift].template as<const float>() : a.t;
        return tb[(int64_t)(my & mask) * ldh + h];
    };
    float t_next = 0.f;
    if constexpr (!FLY) t_next = shipped(0);
    for (int k0 = 0; k0 < cnt; k0 += B) {
        const int nb = min(B, cnt - k0);
        // gathers of the B source rows (a short last batch repeats its last edge; weight 0)
        typename Row4<T>::Raw raw[B];
        static_for<B>([&](auto kk) {
            const int e = k0 + min((int)decltype(kk)::value, nb - 1);
            const T* z;
            if constexpr (ALL)
                z = GlobalPtr<const T>::at(readlane64(row, e));
            else
                z = static_cast<const T*>(a.Z) + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, e) * ld;
            raw[decltype(kk)::value] = load_lane<T, PAD>(z, foff, on);
        });
        loads_sent();
        // scores: lane k of every head group takes edge k0+k
        const bool valid = k < nb;
        float tv = 0.f;
        if constexpr (FLY) {
            // t_j = <a_l, z_j> from the row just gathered; lane k keeps edge k's value
            float cs[B];
            static_for<B>([&](auto kk) {
                float v[4];
                Row4<T>::unpack(raw[decltype(kk)::value], v);
                float c = al[0] * v[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(al[x], v[x], c);
                cs[decltype(kk)::value] = c;
            });
            if constexpr (B == 8 && LPH >= kScatterSumsFrom) {
                tv = group_sums8<LPH>(cs);
            } else {
                static_for<B>([&](auto kk) {
                    const float c = group_all<LPH, OpSum>(cs[decltype(kk)::value]);
                    tv = (k == decltype(kk)::value) ? c : tv;
                });
            }
        } else {
            tv = t_next;
            if (k0 + B < cnt) t_next = shipped(k0 + B);
        }
        const float e2 = valid ? leaky2(fmaf(tv, kLog2e, s2), a.slope) : -INFINITY;
        const float cmax = group_all<LPH, OpMax>(e2);
        if (__builtin_amdgcn_ballot_w64(cmax > st.m2)) {
            const float mn = fmaxf(st.m2, cmax);
            const float c = fast_exp2(st.m2 - mn);    // first edges: exp2(-inf) = 0
            st.l *= c;
#pragma unroll
            for (int x = 0; x < 4; ++x) st.acc[x] *= c;
            st.m2 = mn;
        }
        const float p = fast_exp2(e2 - st.m2);        // 0 for the lanes without an edge
        st.l += p;
        const Spread<LPH> ps(p);
        static_for<B>([&](auto kk) {
            const float pk = ps.template of<decltype(kk)::value>();
            float v[4];
            Row4<T>::unpack(raw[decltype(kk)::value], v);
#pragma unroll
            for (int x = 0; x < 4; ++x) st.acc[x] = fmaf(pk, v[x], st.acc[x]);
        });
    }
}

// The rows of the list, by workgroup `block` of `n_blocks`.
template <typename T, int LPH, int B, bool ALL, bool FLY, bool PAD, int NW = kWavesPerWG>
__device__ inline void fwd_rows(const FwdP& a, const Tabs& tabs, int block, int n_blocks)
{
    static_assert(B <= LPH, "a sub-batch must fit a head group");
    __shared__ float part[NW][kWave][6];
    __shared__ GlobalPtr<const void> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    if constexpr (ALL) {
        if (threadIdx.x < SAR_MAX_BLOCKS) {
            s_Z[threadIdx.x] = tabs.Z[threadIdx.x];
            s_t[threadIdx.x] = tabs.t[threadIdx.x];
        }
        __syncthreads();
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Padded geometry: a launch of fewer than 64/LPH heads leaves whole head groups without a head.
    // Such a group reads what the last head reads (valid memory), speaks for no edge and owns no
    // output: its lanes' `k` matches no slot, so every weight it forms is zero.
    const int h_pos = lane / LPH, k_pos = lane % LPH;
    const bool head_ok = !PAD || h_pos < a.H;
    const int h = head_ok ? h_pos : a.H - 1, k = head_ok ? k_pos : kWave;
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const int foff = PAD ? h * a.D + 4 * k_pos : lane * 4;
    const bool on = PAD ? head_ok && 4 * k_pos < a.D : true;
    T* outp = static_cast<T*>(a.out);
    float al[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FLY) {
        if (on) load_f32<4>(a.a_l + foff, al);
    }

    auto init = [&](FwdState<LPH>& st, int i, bool carry) {
        st.m2 = -INFINITY;
        st.l = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) st.acc[x] = 0.f;
        if constexpr (!ALL) {
            if (carry) {   // state carried from the blocks already aggregated
                st.m2 = a.m[(int64_t)i * ldh + h] * kLog2e;
                st.l = (k == 0) ? a.l[(int64_t)i * ldh + h] : 0.f;
                if (on) load_f32<4>(a.acc + (int64_t)i * ld + foff, st.acc);
            }
        }
    };
    auto finish = [&](FwdState<LPH>& st, int i) {
        const float l = group_all<LPH, OpSum>(st.l);
        if constexpr (ALL) {
            const float inv = l > 0.f ? 1.f / l : 0.f;
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] = st.acc[x] * inv;
                if (a.act == SAR_ACT_RELU) v[x] = fmaxf(v[x], 0.f);
            }
            store_lane<T, PAD>(outp + (int64_t)i * ld, foff, on, v);
            if (k == 0) a.L[(int64_t)i * ldh + h] = l > 0.f ? (st.m2 + fast_log2(l)) * kLn2 : -INFINITY;
        } else {
            if (on) store_f32<4>(a.acc + (int64_t)i * ld + foff, st.acc);
            if (k == 0) {
                a.m[(int64_t)i * ldh + h] = st.m2 * kLn2;
                a.l[(int64_t)i * ldh + h] = l;
            }
        }
    };
    auto edges_at = [&](int at, int end) { return lane < end - at ? a.indices[at + lane] : 0u; };
    // `mine`: edges_at(beg, end); a chunk's edges are read while the one before it is folded
    auto edges = [&](FwdState<LPH>& st, int beg, int end, int step, uint32_t mine, float s2) {
        for (int cb = beg; cb < end; cb += step) {
            const uint32_t next = edges_at(cb + step, end);
            fwd_chunk<T, LPH, B, ALL, FLY, PAD>(st, a, s_Z, s_t, mine, min(kWave, end - cb), foff, on, h, k, s2, al);
            mine = next;
        }
    };

    // Rows at the head of the list are shared by a team of `team` wavefronts, each with its share of the edges.
    auto shared_rows = [&](auto team_c, int64_t r_begin, int64_t r_end, int64_t place) __attribute__((always_inline)) {
        constexpr int team = decltype(team_c)::value, teams = NW / team;
        const int lead = wave / team * team;
        for (int64_t r0 = r_begin + place * teams; r0 < r_end; r0 += (int64_t)n_blocks * teams) {
            const int64_t r = r0 + wave / team;
            const bool have = teams == 1 || r < r_end;
            FwdState<LPH> st;
            int i = 0;
            float l = 0.f;
            if (have) {
                i = __builtin_amdgcn_readfirstlane((int)a.rows[r]);
                init(st, i, wave == lead);
                int beg = a.indptr[i], end = a.indptr[i + 1];
                const float s = a.s[(int64_t)i * ldh + h];
                const int step = row_share(beg, end, wave - lead, team);
                edges(st, beg, end, step, edges_at(beg, end), s * kLog2e);
                l = group_all<LPH, OpSum>(st.l);
#pragma unroll
                for (int x = 0; x < 4; ++x) part[wave][lane][x] = st.acc[x];
                part[wave][lane][4] = st.m2;
                part[wave][lane][5] = l;
            }
            __syncthreads();
            if (have && wave == lead) {
                float m2 = st.m2, lt = l;
                for (int w = lead + 1; w < lead + team; ++w) {
                    const float om = part[w][lane][4], ol = part[w][lane][5];
                    const float mn = fmaxf(m2, om);
                    const float ref = (mn == -INFINITY) ? 0.f : mn;
                    const float ca = fast_exp2(m2 - ref), cb = fast_exp2(om - ref);
                    lt = lt * ca + ol * cb;
#pragma unroll
                    for (int x = 0; x < 4; ++x) st.acc[x] = st.acc[x] * ca + part[w][lane][x] * cb;
                    m2 = mn;
                }
                st.m2 = m2;
                st.l = (k == 0) ? lt : 0.f;
                finish(st, i);
            }
            __syncthreads();
        }
    };
    int64_t hubs = 0;
    if constexpr (NW > kWavesPerWG) {
        hubs = a.n_hub;
        shared_rows(std::integral_constant<int, NW>{}, 0, hubs, block);
    }
    shared_rows(std::integral_constant<int, kWavesPerWG>{}, hubs, a.n_long, from_behind(hubs, block, n_blocks));
    const int64_t n_waves = (int64_t)n_blocks * NW;
    if constexpr (!ALL) {
        // Block by block most of a row is its state, read and written, and the rows are taken one by one.  (As below: bf16 4 x 64 and 8 x
        // 32, 8 blocks of 15 M edges in all, 2103 -> 2230 us, 16 blocks of 0.4 M 274 -> 291; fp32 there 312 -> 328.)
        for (int64_t r = a.n_long + from_behind(a.n_long, block, n_blocks) * NW + wave; r < a.n_rows; r += n_waves) {
            const int i = __builtin_amdgcn_readfirstlane((int)a.rows[r]);
            FwdState<LPH> st;
            init(st, i, true);
            const int beg = a.indptr[i], end = a.indptr[i + 1];
            const float s = a.s[(int64_t)i * ldh + h];
            edges(st, beg, end, kWave, edges_at(beg, end), s * kLog2e);
            finish(st, i);
        }
        return;
    }
    // The other rows, 64 of a wavefront's at a time: lane u reads what there is to know of the u-th (its place in the index),
    // so that a row does not wait for its list entry and then for its range; its first edges and its score half are read while
    // the row before it is folded.  What binds small and middling launches is this chain of loads, not the bytes.  (With the
    // addresses looked up by lanes, 40 layers of 5 us to 31 ms: 7% shorter on average, up to 19; 2 x 128 over 0.3 M edges 74 -> 64
    // us, 8 x 32 over 0.3 M 47 -> 40; those that the memory's rate binds as before, 15 M edges of 1 KiB 2.17 ms.)
    for (int64_t r = a.n_long + from_behind(a.n_long, block, n_blocks) * NW + wave; r < a.n_rows; r += n_waves * kWave) {
        const bool have = r + lane * n_waves < a.n_rows;
        const int count = __builtin_popcountll(__builtin_amdgcn_ballot_w64(have));
        int row = 0, row_beg = 0, row_end = 0;
        if (have) {
            row = (int)a.rows[r + lane * n_waves];
            row_beg = a.indptr[row];
            row_end = a.indptr[row + 1];
        }
        auto of = [&](int v, int u) { return __builtin_amdgcn_readlane(v, u); };
        uint32_t mine = edges_at(of(row_beg, 0), of(row_end, 0));
        float s = a.s[(int64_t)of(row, 0) * ldh + h];
        for (int u = 0; u < count; ++u) {
            const int i = of(row, u), beg = of(row_beg, u), end = of(row_end, u), v = min(u + 1, count - 1);
            const uint32_t mine_next = edges_at(of(row_beg, v), of(row_end, v));
            const float s_next = a.s[(int64_t)of(row, v) * ldh + h];
            FwdState<LPH> st;
            init(st, i, true);
            edges(st, beg, end, kWave, mine, s * kLog2e);
            finish(st, i);
            mine = mine_next;
            s = s_next;
        }
    }
}

// NW: wavefronts of a workgroup.  Two workgroups of twelve fill a CU as far as six of four do, where registers let them.
template <typename T, int LPH, int B, bool FLY, bool PAD, int NW>
__global__ __launch_bounds__(NW * kWave, NW > kWavesPerWG ? 6 : 1) void k_gat_fwd_f256(FwdP a, Tabs tabs)
{
    fwd_rows<T, LPH, B, true, FLY, PAD, NW>(a, tabs, (int)blockIdx.x, (int)gridDim.x);
}

// ----------------------------------------------------------------- backward

struct BwdTabs {
    const int32_t* t_indptr[SAR_MAX_BLOCKS];
    const int32_t* t_indices[SAR_MAX_BLOCKS];
    const void* Z[SAR_MAX_BLOCKS];
    const float* t[SAR_MAX_BLOCKS];
    void* dZ[SAR_MAX_BLOCKS];
    float* dt[SAR_MAX_BLOCKS];
    const int32_t* rank[SAR_MAX_BLOCKS];   // compact outputs: row of dZ / dt that source j owns (null: j itself)
};

struct BwdP {
    const uint32_t* rows;
    int64_t n_rows, n_long;
    const void* G;
    const float4* rec;
    const float* a_l;
    float* ds;           // score gradients of the destinations: the array itself or the first of ds_copies copies
    int64_t ds_stride;   // values between copies
    int ds_copies;       // a power of two; workgroup w adds to copy w % ds_copies
    float* partial;
    int H;
    int tag_shift;
    float slope;
    int ld, ldh, D;      // padded geometry, as in FwdP
};

// The copy of ds this workgroup adds to.
__device__ inline float* ds_of(const BwdP& a)
{
    return a.ds + (int64_t)(blockIdx.x & (unsigned)(a.ds_copies - 1)) * a.ds_stride;
}

// What a lane still has to add to ds.  An atomic addition is performed in memory, never in an L2, and answered a
// microsecond and more later; and the counter by which a wavefront waits for its loads goes down in the order of the
// requests.  Sent as soon as it is known, an addition is waited for with the next batch's rows; so it is sent behind them.
struct DsLater {
    float* to = nullptr;
    float du = 0.f;
    __device__ inline void send()
    {
        if (to) unsafeAtomicAdd(to, du);
        to = nullptr;
    }
    __device__ inline void set(bool valid, float* p, float v)
    {
        to = valid ? p : nullptr;
        du = v;
    }
};

// alpha where `valid`, else 0.  (By bits: a choice of values becomes a branch, and the record's L is then read inside
// it, when the products are done and the rest of the record has long been there.)
__device__ inline float alpha_if(bool valid, float u2, float slope, float L2)
{
    const uint32_t keep = valid ? 0xffffffffu : 0u;
    return __uint_as_float(__float_as_uint(fast_exp2(leaky2(u2, slope) - L2)) & keep);
}

struct BwdAcc4 {
    float dz[4];   // sum_i alpha G_i for the lane's 4 features
    float dt;      // this lane's share of sum_i du
};

template <typename T, int LPH, int B, bool PAD>
__device__ inline void bwd_chunk(BwdAcc4& ac, DsLater& later, const BwdP& a, float* ds, int mine, int cnt, int foff, bool on,
                                 int h, int k, const float (&zj)[4], float t2)
{
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const T* Gp = static_cast<const T*>(a.G);
    for (int k0 = 0; k0 < cnt; k0 += B) {
        const int nb = min(B, cnt - k0);
        typename Row4<T>::Raw raw[B];
        static_for<B>([&](auto kk) {
            const int e = k0 + min((int)decltype(kk)::value, nb - 1);
            const int i = __builtin_amdgcn_readlane(mine, e);
            raw[decltype(kk)::value] = load_lane<T, PAD>(Gp + (int64_t)i * ld, foff, on);
        });
        const bool valid = k < nb;
        const int my_i = __shfl(mine, k0 + (valid ? k : 0));
        const float4 rec = a.rec[(int64_t)my_i * ldh + h];
        later.send();
        loads_sent();
        // c_k = <G_i, z_j> per head, reduced over the head's lanes; lane k keeps edge k's value
        float c_mine = 0.f;
        float cs[B];
        static_for<B>([&](auto kk) {
            float g[4];
            Row4<T>::unpack(raw[decltype(kk)::value], g);
            float c = g[0] * zj[0];
#pragma unroll
            for (int x = 1; x < 4; ++x) c = fmaf(g[x], zj[x], c);
            cs[decltype(kk)::value] = c;
        });
        if constexpr (B == 8 && LPH >= kScatterSumsFrom) {
            c_mine = group_sums8<LPH>(cs);
        } else {
            static_for<B>([&](auto kk) {
                const float c = group_all<LPH, OpSum>(cs[decltype(kk)::value]);
                c_mine = (k == decltype(kk)::value) ? c : c_mine;
            });
        }
        const float u2 = rec.x + t2;
        const float alpha = alpha_if(valid, u2, a.slope, rec.y);
        const float de = alpha * (c_mine - rec.z);
        const float du = u2 > 0.f ? de : a.slope * de;
        ac.dt += du;
        later.set(valid, ds + (int64_t)my_i * ldh + h, du);
        const Spread<LPH> as(alpha);
        static_for<B>([&](auto kk) {
            const float ak = as.template of<decltype(kk)::value>();
            float g[4];
            Row4<T>::unpack(raw[decltype(kk)::value], g);
#pragma unroll
            for (int x = 0; x < 4; ++x) ac.dz[x] = fmaf(ak, g[x], ac.dz[x]);
        });
    }
}

// The wide sources, by workgroup `block` of `n_blocks`; its share of da_l goes to partial_row.
template <typename T, int LPH, int B, bool ALL, bool PAD>
__device__ inline void bwd_wide(const BwdTabs& tabs, const BwdP& a, int block, int n_blocks, float* partial_row)
{
    static_assert(B <= LPH, "a sub-batch must fit a head group");
    __shared__ float part[kWavesPerWG][kWave][5];
    __shared__ GlobalPtr<const void> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<void> s_dZ[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<float> s_dt[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ip[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ix[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_rank[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_Z[threadIdx.x] = tabs.Z[threadIdx.x];
        s_t[threadIdx.x] = tabs.t[threadIdx.x];
        s_dZ[threadIdx.x] = tabs.dZ[threadIdx.x];
        s_dt[threadIdx.x] = tabs.dt[threadIdx.x];
        s_ip[threadIdx.x] = tabs.t_indptr[threadIdx.x];
        s_ix[threadIdx.x] = tabs.t_indices[threadIdx.x];
        s_rank[threadIdx.x] = tabs.rank[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Padded geometry: a launch of fewer than 64/LPH heads leaves whole head groups without a head.
    // Such a group reads what the last head reads (valid memory), speaks for no edge and owns no
    // output: its lanes' `k` matches no slot, so every weight it forms is zero.
    const int h_pos = lane / LPH, k_pos = lane % LPH;
    const bool head_ok = !PAD || h_pos < a.H;
    const int h = head_ok ? h_pos : a.H - 1, k = head_ok ? k_pos : kWave;
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const int foff = PAD ? h * a.D + 4 * k_pos : lane * 4;
    const bool on = PAD ? head_ok && 4 * k_pos < a.D : true;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;

    float* const ds = ds_of(a);
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4];
    if (on) load_f32<4>(a.a_l + foff, al);
#pragma unroll
    for (int x = 0; x < 4; ++x) dal[x] = 0.f;

    // What there is to know of a source: the addresses of its row and of its error's, its edges' destinations.
    struct Src {
        uint32_t id;
        int row_out, count;
        uint64_t z, dst;
    };
    auto source = [&](uint32_t id) {
        const int q = ALL ? (int)(id >> a.tag_shift) : 0, j = (int)(id & mask);
        const int beg = s_ip[q][j];
        Src x{id, s_rank[q] ? s_rank[q][j] : j, s_ip[q][j + 1] - beg, 0, 0};
        x.z = s_Z[q].bits + (uint64_t)j * (uint32_t)(ld * (int)sizeof(T));
        x.dst = s_ix[q].bits + (uint64_t)beg * sizeof(int32_t);
        return x;
    };
    auto load_z = [&](uint64_t z) { return load_lane<T, PAD>(GlobalPtr<const T>::at(z), foff, on); };
    auto edges_at = [&](uint64_t dst, int at, int end) {
        const int32_t* const i = GlobalPtr<const int32_t>::at(dst);
        return lane < end - at ? i[at + lane] : 0;
    };
    DsLater later;
    // the source's edges [beg, end); `mine`: edges_at(dst, beg, end)
    auto edges = [&](BwdAcc4& ac, uint32_t id, uint64_t dst, int beg, int end, int step, int mine, const float (&zj)[4]) {
        const int q = ALL ? (int)(id >> a.tag_shift) : 0;
        float t2;
        if (s_t[q]) {
            t2 = score_log2(s_t[q][(int64_t)(id & mask) * ldh + h]);
        } else {   // t_j = <a_l, z_j> from the row this wavefront owns
            float c = al[0] * zj[0];
#pragma unroll
            for (int x = 1; x < 4; ++x) c = fmaf(al[x], zj[x], c);
            t2 = score_log2(group_all<LPH, OpSum>(c));
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) ac.dz[x] = 0.f;
        ac.dt = 0.f;
        for (int cb = beg; cb < end; cb += step) {
            const int next = edges_at(dst, cb + step, end);
            bwd_chunk<T, LPH, B, PAD>(ac, later, a, ds, mine, min(kWave, end - cb), foff, on, h, k, zj, t2);
            mine = next;
        }
    };
    // dZ_q[j] = sum alpha G + dt a_l ; dt_q[j] = dt ; da_l += dt z_j
    auto outputs = [&](const BwdAcc4& ac, float dt, uint32_t id, int64_t jo, const float (&zj)[4]) {
        const int q = ALL ? (int)(id >> a.tag_shift) : 0;
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            v[x] = fmaf(dt, al[x], ac.dz[x]);
            dal[x] = fmaf(dt, zj[x], dal[x]);
        }
        store_lane<T, PAD>(s_dZ[q].template as<T>() + jo * ld, foff, on, v);
        if (k == 0 && s_dt[q]) s_dt[q][jo * ldh + h] = dt;
    };

    for (int64_t r = block; r < a.n_long; r += n_blocks) {
        const Src x = source(a.rows[r]);
        BwdAcc4 ac;
        float zj[4];
        int beg = 0, end = x.count;
        const int step = row_share(beg, end, wave, kWavesPerWG);
        const int mine = edges_at(x.dst, beg, end);
        Row4<T>::unpack(load_z(x.z), zj);
        edges(ac, x.id, x.dst, beg, end, step, mine, zj);
        const float dt = group_all<LPH, OpSum>(ac.dt);
#pragma unroll
        for (int x = 0; x < 4; ++x) part[wave][lane][x] = ac.dz[x];
        part[wave][lane][4] = dt;
        __syncthreads();
        if (wave == 0) {
            float tot[5];
#pragma unroll
            for (int x = 0; x < 5; ++x) {
                float s = 0.f;
                for (int w = 0; w < kWavesPerWG; ++w) s += part[w][lane][x];
                tot[x] = s;
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) ac.dz[x] = tot[x];
            outputs(ac, tot[4], x.id, x.row_out, zj);
        }
        __syncthreads();
    }
    // The other sources, 64 of a wavefront's at a time: lane u looks up the u-th, and its own row and first destinations are
    // read while the source before it is taken.  (With the record read at once and the additions sent late, 40 layers of 6 us to
    // 36 ms: 13% shorter on average, up to 34; 2 x 100 bf16 block by block 167 -> 111 us, 4 x 64 bf16 over 3 M edges 238 -> 213.)
    const int64_t n_waves = (int64_t)n_blocks * kWavesPerWG;
    for (int64_t r = a.n_long + from_behind(a.n_long, block, n_blocks) * kWavesPerWG + wave; r < a.n_rows;
         r += n_waves * kWave) {
        const bool have = r + lane * n_waves < a.n_rows;
        const int count = __builtin_popcountll(__builtin_amdgcn_ballot_w64(have));
        Src x{0, 0, 0, 0, 0};
        if (have) x = source(a.rows[r + lane * n_waves]);
        auto of = [&](int v, int u) { return __builtin_amdgcn_readlane(v, u); };
        typename Row4<T>::Raw zr = load_z(readlane64(x.z, 0));
        int mine = edges_at(readlane64(x.dst, 0), 0, of(x.count, 0));
        for (int u = 0; u < count; ++u) {
            const int v = min(u + 1, count - 1);
            float zj[4];
            Row4<T>::unpack(zr, zj);
            zr = load_z(readlane64(x.z, v));
            const int mine_next = edges_at(readlane64(x.dst, v), 0, of(x.count, v));
            BwdAcc4 ac;
            const uint32_t id = (uint32_t)of((int)x.id, u);
            edges(ac, id, readlane64(x.dst, u), 0, of(x.count, u), kWave, mine, zj);
            outputs(ac, group_all<LPH, OpSum>(ac.dt), id, of(x.row_out, u), zj);
            mine = mine_next;
        }
    }
    later.send();

    // this workgroup's share of da_l = sum_j dt_j z_j
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) part[wave][lane][x] = dal[x];
    __syncthreads();
    if (wave == 0) {
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float s = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) s += part[w][lane][x];
            v[x] = s;
        }
        store_f32<4>(partial_row + lane * 4, v);
    }
}

template <typename T, int LPH, int B, bool ALL, bool PAD>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd_f256(BwdTabs tabs, BwdP a)
{
    bwd_wide<T, LPH, B, ALL, PAD>(tabs, a, (int)blockIdx.x, (int)gridDim.x, a.partial + (int64_t)blockIdx.x * kF);
}

// ------------------------------------------- backward, rows of few edges
//
// A source of fewer than 8 edges would leave most of a wide-kernel batch empty.  This kernel
// keeps the lane geometry of the wide kernel -- lane x owns
// features 4x..4x+3 of every row, so each row -- a source's own row, a gathered G row, the error
// row written back -- is one fully coalesced wave-wide access.  Independent work comes from
// taking S sources per wavefront at once: a round gathers B = S*R rows, R edges of each of the
// S sources, and lane k of every head group speaks for gather slot k (the edge's record,
// coefficient and score gradient), exactly as it speaks for edge k of a sub-batch in the wide
// kernel; slot k always belongs to source k / R, so a lane's share of dt needs no indexing.
//
// What describes a source is read ahead by the lanes themselves, one register per field:
// lane u*kAhead + e holds source u's list entry, edge range and output row, and the
// destination of its edge e.  List entries are read three groups ahead, ranges two, and
// destinations one, so that a group starts with its row gathers and no dependent chain.
template <typename T, int LPH, bool ALL, bool PAD>
__device__ inline void bwd_few(const BwdTabs& tabs, const BwdP& a, int64_t r_begin, int64_t r_end, int block, int n_blocks,
                               float* partial_row)
{
    constexpr int B = LPH >= 8 ? 8 : 4;   // gather slots per round
    constexpr int R = 2;                  // slots per source
    constexpr int S = B / R;              // sources per wavefront and group
    constexpr int kAhead = 8;             // edges per source whose destinations are read ahead: all of them
    static_assert(S * kAhead <= kWave, "one lane per (source, edge read ahead)");
    static_assert((1 << kNarrowMaxClass) <= kAhead, "this kernel's sources have fewer than kAhead edges");
    __shared__ float part[kWavesPerWG][kWave][4];
    __shared__ GlobalPtr<const void> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<void> s_dZ[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<float> s_dt[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ip[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ix[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_rank[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_Z[threadIdx.x] = tabs.Z[threadIdx.x];
        s_t[threadIdx.x] = tabs.t[threadIdx.x];
        s_dZ[threadIdx.x] = tabs.dZ[threadIdx.x];
        s_dt[threadIdx.x] = tabs.dt[threadIdx.x];
        s_ip[threadIdx.x] = tabs.t_indptr[threadIdx.x];
        s_ix[threadIdx.x] = tabs.t_indices[threadIdx.x];
        s_rank[threadIdx.x] = tabs.rank[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // exact geometry: rows of 256 values; padded: heads of any width D <= 4 LPH inside rows of stride
    // ld, head groups beyond the launch's heads idle (see k_gat_fwd_f256)
    const int h_pos = lane / LPH, k_pos = lane % LPH;
    const bool head_ok = !PAD || h_pos < a.H;
    const int h = head_ok ? h_pos : a.H - 1, k = head_ok ? k_pos : kWave;
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const int foff = PAD ? h * a.D + 4 * k_pos : lane * 4;
    const bool on = PAD ? head_ok && 4 * k_pos < a.D : true;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    const T* Gp = static_cast<const T*>(a.G);

    float* const ds = ds_of(a);
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4];
    if (on) load_f32<4>(a.a_l + foff, al);
#pragma unroll
    for (int x = 0; x < 4; ++x) dal[x] = 0.f;

    // ---- the lanes' read-ahead of list entries, ranges and destinations
    const bool meta_lane = lane < S * kAhead;
    const int mu = lane / kAhead, me = lane % kAhead;
    const int64_t stride = (int64_t)n_blocks * kWavesPerWG * S;
    struct Range { int q, j, beg, end, jo; };
    auto valid = [&](int64_t g) { return meta_lane && g + mu < r_end; };
    auto load_id = [&](int64_t g) -> uint32_t { return valid(g) ? a.rows[g + mu] : 0u; };
    auto load_range = [&](uint32_t id, int64_t g) {
        Range m{0, 0, 0, 0, 0};
        if (valid(g)) {
            m.q = ALL ? (int)(id >> a.tag_shift) : 0;
            m.j = (int)(id & mask);
            const int32_t* ip = s_ip[m.q];
            m.beg = ip[m.j];
            m.end = ip[m.j + 1];
            m.jo = s_rank[m.q] ? s_rank[m.q][m.j] : m.j;
        }
        return m;
    };
    auto load_dst = [&](const Range& m, int64_t g) { return (valid(g) && me < m.end - m.beg) ? s_ix[m.q][m.beg + me] : 0; };

    int64_t g0 = r_begin + ((int64_t)block * kWavesPerWG + wave) * S;
    uint32_t id2 = load_id(g0 + 2 * stride);
    Range m0 = load_range(load_id(g0), g0), m1 = load_range(load_id(g0 + stride), g0 + stride);
    int dst0 = load_dst(m0, g0);

    for (; g0 < r_end; g0 += stride) {
        const int dst1 = load_dst(m1, g0 + stride);
        const Range m2 = load_range(id2, g0 + 2 * stride);
        const uint32_t id3 = load_id(g0 + 3 * stride);

        // ---- the S sources of this group: uniform values out of the lanes that hold them
        bool have[S];
        int q[S], j[S], beg[S], end[S], jo[S];
        typename Row4<T>::Raw zr[S];
        int rounds = 0;
        static_for<S>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            have[u] = g0 + u < r_end;
            q[u] = __builtin_amdgcn_readlane(m0.q, u * kAhead);
            j[u] = __builtin_amdgcn_readlane(m0.j, u * kAhead);
            beg[u] = __builtin_amdgcn_readlane(m0.beg, u * kAhead);
            end[u] = __builtin_amdgcn_readlane(m0.end, u * kAhead);
            jo[u] = __builtin_amdgcn_readlane(m0.jo, u * kAhead);
            rounds = max(rounds, end[u] - beg[u]);
            zr[u] = typename Row4<T>::Raw{};
            if (have[u]) zr[u] = load_lane<T, PAD>(s_Z[q[u]].template as<const T>() + (int64_t)j[u] * ld, foff, on);
        });
        float t2[S], dz[S][4];
        static_for<S>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
#pragma unroll
            for (int x = 0; x < 4; ++x) dz[u][x] = 0.f;
            t2[u] = 0.f;
            if (have[u]) {
                if (s_t[q[u]]) {
                    t2[u] = score_log2(s_t[q[u]][(int64_t)j[u] * ldh + h]);
                } else {   // t_j = <a_l, z_j> from the row this wavefront holds
                    float zj[4];
                    Row4<T>::unpack(zr[u], zj);
                    float c = al[0] * zj[0];
#pragma unroll
                    for (int x = 1; x < 4; ++x) c = fmaf(al[x], zj[x], c);
                    t2[u] = score_log2(group_all<LPH, OpSum>(c));
                }
            }
        });
        // the source this lane's slot belongs to
        float t2_mine = t2[0];
        static_for<S>([&](auto uu) { t2_mine = (k / R == decltype(uu)::value) ? t2[decltype(uu)::value] : t2_mine; });
        float dt_mine = 0.f;

        for (int e = 0; e < rounds; e += R) {
            int dst[B];
            bool ok[B];
            typename Row4<T>::Raw raw[B];
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value, u = K / R, r = K % R;
                ok[K] = beg[u] + e + r < end[u];
                dst[K] = 0;
                raw[K] = typename Row4<T>::Raw{};
                if (ok[K]) dst[K] = __builtin_amdgcn_readlane(dst0, u * kAhead + e + r);
            });
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                if (ok[K]) raw[K] = load_lane<T, PAD>(Gp + (int64_t)dst[K] * ld, foff, on);
            });
            // lane k speaks for slot k
            int my_i = 0;
            bool my_ok = false;
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                my_i = (k == K) ? dst[K] : my_i;
                my_ok = (k == K) ? ok[K] : my_ok;
            });
            float4 rec = make_float4(0.f, INFINITY, 0.f, 0.f);   // L = +inf gives alpha = 0
            if (my_ok) rec = a.rec[(int64_t)my_i * ldh + h];
            loads_sent();
            float c_mine = 0.f;
            float cs[B];
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                float g[4], zj[4];
                Row4<T>::unpack(raw[K], g);
                Row4<T>::unpack(zr[K / R], zj);
                float c = g[0] * zj[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(g[x], zj[x], c);
                cs[K] = c;
            });
            if constexpr (B == 8 && LPH >= kScatterSumsFrom) {
                c_mine = group_sums8<LPH>(cs);
            } else {
                static_for<B>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const float c = group_all<LPH, OpSum>(cs[K]);
                    c_mine = (k == K) ? c : c_mine;
                });
            }
            const float u2 = rec.x + t2_mine;
            const float alpha = alpha_if(my_ok, u2, a.slope, rec.y);
            const float de = alpha * (c_mine - rec.z);
            const float du = u2 > 0.f ? de : a.slope * de;
            dt_mine += du;
            if (my_ok) unsafeAtomicAdd(ds + (int64_t)my_i * ldh + h, du);
            const Spread<LPH> as(alpha);
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float ak = as.template of<K>();
                float g[4];
                Row4<T>::unpack(raw[K], g);
#pragma unroll
                for (int x = 0; x < 4; ++x) dz[K / R][x] = fmaf(ak, g[x], dz[K / R][x]);
            });
        }

        // ---- dZ_q[j] = sum alpha G + dt a_l ; dt_q[j] = dt ; da_l += dt z_j
        const Spread<LPH> dts(dt_mine);
        static_for<S>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            float dt = 0.f;
            static_for<R>([&](auto rr) { dt += dts.template of<u * R + decltype(rr)::value>(); });
            if (have[u]) {
                float v[4], zj[4];
                Row4<T>::unpack(zr[u], zj);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = fmaf(dt, al[x], dz[u][x]);
                    dal[x] = fmaf(dt, zj[x], dal[x]);
                }
                store_lane<T, PAD>(s_dZ[q[u]].template as<T>() + (int64_t)jo[u] * ld, foff, on, v);
                if (k == 0 && s_dt[q[u]]) s_dt[q[u]][(int64_t)jo[u] * ldh + h] = dt;
            }
        });
        m0 = m1;
        dst0 = dst1;
        m1 = m2;
        id2 = id3;
    }

    // this workgroup's share of da_l
#pragma unroll
    for (int x = 0; x < 4; ++x) part[wave][lane][x] = dal[x];
    __syncthreads();
    if (wave == 0) {
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float s = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) s += part[w][lane][x];
            v[x] = s;
        }
        store_f32<4>(partial_row + lane * 4, v);
    }
}

template <typename T, int LPH, bool ALL, bool PAD>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd_few(BwdTabs tabs, BwdP a, int64_t r_begin, int64_t r_end,
                                                                int partial_row0)
{
    bwd_few<T, LPH, ALL, PAD>(tabs, a, r_begin, r_end, (int)blockIdx.x, (int)gridDim.x,
                              a.partial + ((int64_t)partial_row0 + blockIdx.x) * kF);
}

// ------------------------------------------- backward, sources of one edge
//
// A source with ONE edge in its block gains nothing from being walked source-major: its own row,
// its error row, and a gathered row of G with that destination's record, for one edge.  This
// kernel takes such edges in the order of their DESTINATIONS (a list the builder derives from the
// all-blocks index): the entries of a destination follow each other, so its row of G and its
// record come from the caches after the first of them, and what is left per edge is the source's
// row and one write of its error row -- which nobody else writes, so dZ_q[j] = alpha G_i + du a_l
// and dt_q[j] = du are plain stores.  Lane geometry and the sub-batch of B gather slots are those
// of the wide kernel; slot k here is an (edge, source) of its own and lane k of every head group
// speaks for it.
struct SingleP {
    const int32_t* dst;    // [n] destination of the entry's edge
    const uint32_t* src;   // [n] its source, tagged with the block
    const int32_t* row;    // [n] row of the source in its block's dZ_q / dt_q
    int64_t n;
    int per;               // entries a wavefront takes at a time, at most 64
};

template <typename T, int LPH, bool PAD>
__device__ inline void bwd_single(const BwdTabs& tabs, const BwdP& a, const SingleP& s, int block, int n_blocks,
                                  float* partial_row)
{
    constexpr int B = LPH >= 8 ? 8 : 4;
    static_assert(B <= LPH, "a sub-batch must fit a head group");
    __shared__ float part[kWavesPerWG][kWave][4];
    __shared__ GlobalPtr<const void> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<void> s_dZ[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<float> s_dt[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_Z[threadIdx.x] = tabs.Z[threadIdx.x];
        s_t[threadIdx.x] = tabs.t[threadIdx.x];
        s_dZ[threadIdx.x] = tabs.dZ[threadIdx.x];
        s_dt[threadIdx.x] = tabs.dt[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // exact geometry: rows of 256 values; padded: heads of any width D <= 4 LPH inside rows of stride
    // ld, head groups beyond the launch's heads idle (see k_gat_fwd_f256)
    const int h_pos = lane / LPH, k_pos = lane % LPH;
    const bool head_ok = !PAD || h_pos < a.H;
    const int h = head_ok ? h_pos : a.H - 1, k = head_ok ? k_pos : kWave;
    const int ld = PAD ? a.ld : kF, ldh = PAD ? a.ldh : a.H;
    const int foff = PAD ? h * a.D + 4 * k_pos : lane * 4;
    const bool on = PAD ? head_ok && 4 * k_pos < a.D : true;
    const uint32_t mask = (1u << a.tag_shift) - 1u;
    const T* Gp = static_cast<const T*>(a.G);

    float* const ds = ds_of(a);
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4];
    if (on) load_f32<4>(a.a_l + foff, al);
#pragma unroll
    for (int x = 0; x < 4; ++x) dal[x] = 0.f;

    // a wavefront takes `per` entries at a time, one per lane; the next ones travel meanwhile
    const int64_t n_chunks = (s.n + s.per - 1) / s.per;
    const int64_t stride = (int64_t)n_blocks * kWavesPerWG;
    struct Entry { int i; uint32_t id; int row; };
    auto load_entries = [&](int64_t c) {
        Entry e{0, 0u, 0};
        const int64_t at = c * s.per + lane;
        if (c < n_chunks && lane < s.per && at < s.n) e = Entry{s.dst[at], s.src[at], s.row[at]};
        return e;
    };
    int64_t c = (int64_t)block * kWavesPerWG + wave;
    Entry cur = load_entries(c);
    for (; c < n_chunks; c += stride) {
        const Entry nxt = load_entries(c + stride);
        const int cnt = (int)min((int64_t)s.per, s.n - c * s.per);
        for (int k0 = 0; k0 < cnt; k0 += B) {
            const int nb = min(B, cnt - k0);
            int q[B], row[B];
            typename Row4<T>::Raw rg[B], rz[B];
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const int e = k0 + min(K, nb - 1);
                const int i = __builtin_amdgcn_readlane(cur.i, e);
                const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)cur.id, e);
                q[K] = (int)(id >> a.tag_shift);
                row[K] = __builtin_amdgcn_readlane(cur.row, e);
                rg[K] = load_lane<T, PAD>(Gp + (int64_t)i * ld, foff, on);
                rz[K] = load_lane<T, PAD>(s_Z[q[K]].template as<const T>() + (int64_t)(id & mask) * ld, foff, on);
            });
            // lane k speaks for slot k
            const bool valid = k < nb;
            const int sel = k0 + (valid ? k : 0);
            const int my_i = __shfl(cur.i, sel);
            const uint32_t my_id = (uint32_t)__shfl((int)cur.id, sel);
            const int my_row = __shfl(cur.row, sel);
            const int my_q = (int)(my_id >> a.tag_shift);
            const float4 rec = a.rec[(int64_t)my_i * ldh + h];
            loads_sent();
            float cs[B], ts[B];
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                float g[4], z[4];
                Row4<T>::unpack(rg[K], g);
                Row4<T>::unpack(rz[K], z);
                float cg = g[0] * z[0], ct = al[0] * z[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) {
                    cg = fmaf(g[x], z[x], cg);
                    ct = fmaf(al[x], z[x], ct);
                }
                cs[K] = cg;
                ts[K] = ct;
            });
            float c_mine = 0.f, t_mine = 0.f;
            if constexpr (B == 8 && LPH >= kScatterSumsFrom) {
                c_mine = group_sums8<LPH>(cs);
                t_mine = group_sums8<LPH>(ts);
            } else {
                static_for<B>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const float cg = group_all<LPH, OpSum>(cs[K]);
                    const float ct = group_all<LPH, OpSum>(ts[K]);
                    c_mine = (k == K) ? cg : c_mine;
                    t_mine = (k == K) ? ct : t_mine;
                });
            }
            if (valid && s_t[my_q]) t_mine = s_t[my_q][(int64_t)(my_id & mask) * ldh + h];
            const float u2 = rec.x + score_log2(t_mine);
            const float alpha = alpha_if(valid, u2, a.slope, rec.y);
            const float de = alpha * (c_mine - rec.z);
            const float du = u2 > 0.f ? de : a.slope * de;
            if (valid && s_dt[my_q]) s_dt[my_q][(int64_t)my_row * ldh + h] = du;
            // ds_i += du: the entries of a destination follow each other, and a frequent destination
            // fills whole sub-batches: one atomic per run of slots that share the destination
            // (a running sum along the run, added by its last slot), not one per slot on one address
            {
                const int seg = valid ? my_i : -1 - k;
                float run = du;
                static_for<3>([&](auto ss) {
                    constexpr int sh = 1 << decltype(ss)::value;
                    if constexpr (sh < B) {
                        const float r_s = dpp<kRowShr + sh>(run);
                        const int i_s = dpp_i<kRowShr + sh>(seg);
                        if (k >= sh && i_s == seg) run += r_s;
                    }
                });
                const int next = dpp_i<kRowShl + 1>(seg);
                if (valid && (k == B - 1 || next != seg)) unsafeAtomicAdd(ds + (int64_t)my_i * ldh + h, run);
            }
            const Spread<LPH> as(alpha), us(du);
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float ak = as.template of<K>();
                const float dk = us.template of<K>();
                float g[4], z[4], v[4];
                Row4<T>::unpack(rg[K], g);
                Row4<T>::unpack(rz[K], z);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = fmaf(dk, al[x], ak * g[x]);
                    dal[x] = fmaf(dk, z[x], dal[x]);
                }
                if (K < nb) store_lane<T, PAD>(s_dZ[q[K]].template as<T>() + (int64_t)row[K] * ld, foff, on, v);
            });
        }
        cur = nxt;
    }

    // this workgroup's share of da_l
#pragma unroll
    for (int x = 0; x < 4; ++x) part[wave][lane][x] = dal[x];
    __syncthreads();
    if (wave == 0) {
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float sum = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) sum += part[w][lane][x];
            v[x] = sum;
        }
        store_f32<4>(partial_row + lane * 4, v);
    }
}

template <typename T, int LPH, bool PAD>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd_single(BwdTabs tabs, BwdP a, SingleP s, int partial_row0)
{
    bwd_single<T, LPH, PAD>(tabs, a, s, (int)blockIdx.x, (int)gridDim.x,
                            a.partial + ((int64_t)partial_row0 + blockIdx.x) * kF);
}

}  // namespace f256
}  // namespace sar
