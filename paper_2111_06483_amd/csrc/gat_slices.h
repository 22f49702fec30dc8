// Attention kernels for dense graphs: every XCD gathers one head's slice of the rows.
//
// A row of H heads is read by every edge that cites it.  Where rows have hundreds of edges and no row is a hub, the
// kernels of gat_f256.h take each of those reads from memory: the rows in use at a time do not fit in an XCD's 4 MiB of
// L2.  Here workgroup b serves head b % 8, and workgroups are dealt to the eight XCDs in that order, so that an XCD's L2
// holds slices of one head only; and a lane group of LPH = D/4 lanes owns a row of its own, so that 64/LPH rows a
// wavefront, a thousand an XCD with 32 lanes a row, are walked at a time.  Their edges are sorted by source and the
// rows by number of edges, so at any time the rows of an XCD are at about the same place of the source list: they sweep
// over it together, a slice is fetched once a sweep and the other rows that cite it find it in L2.
// (Performance only: nothing depends on where a workgroup runs.)
//
// The arithmetic of a row is that of gat_f256.h, batch by batch and lane by lane: the same bits where one wavefront walks
// the row there (256 values, fewer edges than workgroups share).
#pragma once

#include "gat_f256.h"

namespace sar {
namespace slices {

using f256::dpp;
using f256::FwdP;
using f256::group_all;
using f256::leaky2;
using f256::load_lane;
using f256::OpMax;
using f256::OpSum;
using f256::Row4;
using f256::Spread;
using f256::static_for;
using f256::store_lane;
using f256::Tabs;

constexpr int kXcds = 8;
constexpr int kBatch = 8;    // edges of a row in flight
constexpr int kTurns = 4;    // batches between barriers

// SYNC: workgroups of 16 wavefronts that meet at a barrier every few batches.  A wavefront for itself falls behind or
// runs ahead (older ones are served first), and the sweep comes apart within one pass.  Where the head's slices of the
// whole table fit in L2 there is nothing to keep together, and small workgroups run freely.
template <bool SYNC>
constexpr int kThreads = SYNC ? 1024 : 256;
template <bool SYNC>
constexpr int kWaves = kThreads<SYNC> / kWave;

// Which heads (HS of them) and which share of the rows a workgroup serves.
template <bool SYNC>
struct Unit {
    int set, sets, parts, part, wg, n_wgs;   // its first set of heads; the rows' shares; this workgroup among its unit's
    __device__ inline Unit(int sets_)
    {
        const int unit = blockIdx.x % kXcds;
        sets = sets_;
        parts = sets < kXcds ? kXcds / sets : 1;
        set = unit % (sets < kXcds ? sets : kXcds);
        part = unit / (sets < kXcds ? sets : kXcds);
        wg = (int)(blockIdx.x / kXcds);
        n_wgs = (int)(gridDim.x / kXcds);
    }
    // first row of the workgroup's (of this wavefront's) next turn, and from turn to turn
    __device__ inline int64_t first(int wave, int slots) const
    {
        return ((int64_t)(wg * kWaves<SYNC> + wave) * parts + part) * slots;
    }
    __device__ inline int64_t stride(int slots) const { return (int64_t)n_wgs * kWaves<SYNC> * parts * slots; }
};

// Whether any row of the wavefront (SYNC: of the workgroup, asked every kTurns batches) has edges left.
template <bool SYNC>
__device__ inline bool go_on(bool left, int turn)
{
    if constexpr (SYNC) return turn % kTurns != 0 || __syncthreads_or(left);
    return __builtin_amdgcn_ballot_w64(left) != 0;
}

// Edges of a batch behind a row's end (its last one again) hold zeros: weight 0 alone would turn an infinity of theirs into
// a NaN.  (Most batches have none: one test each.  25 M edges, 8 x 32 fp32: forward 2176 -> 2197 us; batches that lie
// behind the end as a whole are left out, which they were not: backward 3342 -> 3168.)
template <int B, typename Raw>
__device__ inline void zero_behind(Raw (&raw)[B], int left)
{
    if (__builtin_amdgcn_ballot_w64(left < B) == 0) return;
    static_for<B>([&](auto kk) {
        constexpr int K = decltype(kk)::value;
        if (K >= left) raw[K] = Raw{};
    });
}

// ------------------------------------------------------------------ forward, all blocks

template <typename T, int LPH, bool FLY, bool PAD, bool SYNC>
__global__ __launch_bounds__(kThreads<SYNC>) void k_gat_fwd_slices(FwdP a, Tabs tabs)
{
    constexpr int B = kBatch, kSlots = kWave / LPH;
    static_assert(B <= LPH, "a batch must fit a head group");
    __shared__ GlobalPtr<const T> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_Z[threadIdx.x] = static_cast<const T*>(tabs.Z[threadIdx.x]);
        s_t[threadIdx.x] = tabs.t[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = lane / LPH, k = lane % LPH;
    const bool on = !PAD || 4 * k < a.D;
    const uint32_t mask = (1u << a.tag_shift) - 1u;
    const Unit<SYNC> u(a.H);
    for (int h = u.set; h < a.H; h += kXcds) {
        const int foff = h * a.D + (on ? 4 * k : 0);
        float al[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (FLY) {
            if (on) load_f32<4>(a.a_l + foff, al);
        }
        // (SYNC: the wavefronts of a workgroup take as many turns as its first one)
        int64_t r0 = u.first(wave, kSlots);
        for (int64_t w0 = SYNC ? u.first(0, kSlots) : r0; w0 < a.n_rows; w0 += u.stride(kSlots), r0 += u.stride(kSlots)) {
            // (a slot behind the list's end takes the last row again and keeps quiet)
            const bool live = r0 + slot < a.n_rows;
            const int i = (int)a.rows[live ? r0 + slot : a.n_rows - 1];
            const int first = a.indptr[i], len = a.indptr[i + 1] - first;
            const int beg = len > 0 ? first : 0, last = max(len - 1, 0);
            const float s2 = a.s[(int64_t)i * a.ldh + h] * kLog2e;
            float m2 = -INFINITY, l = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
            // lane k of the group reads edge e0 + k (behind the row's end its last edge again, with weight 0; a row without
            // edges the first of the index)
            uint32_t mine = a.indices[beg + min(k, last)];
            for (int e0 = 0, turn = 0; go_on<SYNC>(e0 < len, turn); e0 += B, ++turn) {
                if (e0 >= len) continue;          // (the rows beside this one go on)
                const uint32_t next = a.indices[beg + min(e0 + B + k, last)];
                const int64_t at = (int64_t)(mine & mask);
                const uint64_t row = s_Z[mine >> a.tag_shift].bits + (uint64_t)(at * a.ld) * sizeof(T);
                typename Row4<T>::Raw raw[B];
                const Spread<LPH, LPH <= 32> lo((uint32_t)row), hi((uint32_t)(row >> 32));
                static_for<B>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const uint64_t from = (uint64_t)(uint32_t)lo.template of_int<K>() |
                                          (uint64_t)(uint32_t)hi.template of_int<K>() << 32;
                    raw[K] = load_lane<T, PAD>(GlobalPtr<const T>::at(from), foff, on);
                });
                loads_sent();
                zero_behind(raw, len - e0);
                const bool valid = k < B && e0 + k < len;
                float tv = 0.f;
                if constexpr (FLY) {
                    static_for<B>([&](auto kk) {
                        constexpr int K = decltype(kk)::value;
                        float v[4];
                        Row4<T>::unpack(raw[K], v);
                        float c = al[0] * v[0];
#pragma unroll
                        for (int x = 1; x < 4; ++x) c = fmaf(al[x], v[x], c);
                        c = group_all<LPH, OpSum>(c);
                        tv = k == K ? c : tv;
                    });
                } else {
                    tv = s_t[mine >> a.tag_shift][at * a.ldh + h];
                }
                const float e2 = valid ? leaky2(fmaf(tv, kLog2e, s2), a.slope) : -INFINITY;
                const float cmax = group_all<LPH, OpMax>(e2);
                if (__builtin_amdgcn_ballot_w64(cmax > m2)) {
                    const float mn = fmaxf(m2, cmax);
                    const float c = fast_exp2(m2 - mn);
                    l *= c;
#pragma unroll
                    for (int x = 0; x < 4; ++x) acc[x] *= c;
                    m2 = mn;
                }
                const float p = fast_exp2(e2 - m2);
                l += p;
                const Spread<LPH, LPH <= 32> ps(p);
                static_for<B>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const float pk = ps.template of<K>();
                    float v[4];
                    Row4<T>::unpack(raw[K], v);
#pragma unroll
                    for (int x = 0; x < 4; ++x) acc[x] = fmaf(pk, v[x], acc[x]);
                });
                mine = next;
            }
            l = group_all<LPH, OpSum>(l);
            const float inv = l > 0.f ? 1.f / l : 0.f;
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] = acc[x] * inv;
                if (a.act == SAR_ACT_RELU) v[x] = fmaxf(v[x], 0.f);
            }
            if (live) {
                store_lane<T, PAD>(static_cast<T*>(a.out) + (int64_t)i * a.ld, foff, on, v);
                if (k == 0) a.L[(int64_t)i * a.ldh + h] = l > 0.f ? (m2 + fast_log2(l)) * kLn2 : -INFINITY;
            }
        }
    }
}

// ------------------------------------------------------------------ backward, all blocks
//
// The sources of at least 8 edges, source by source as in k_gat_bwd_f256, a slice being HS heads of 128 values together; one
// or two slices to a row.
// What is added to ds costs more than what is read here: the chip takes some 20 additions a nanosecond, one for every
// edge and set of heads (one head of 32 values at a time, 8 sets: 5.1 ms for 25M edges, fp32 and bf16 alike, where the
// rows take 2 ms), and a destination's record is a request to L2 of its own as well.  So slices are as wide as lets the
// rows of an XCD still sweep G together, and records and ds are laid out by sets, [H / HS][n][HS], in the caller's
// scratch (k_slices_begin, k_slices_end).
struct SetP {
    const float4* rec;   // [H / HS][n_dst][HS]
    float* ds;           // [H / HS][n_dst][HS]
    int64_t n_dst;
};

template <int HS>
__global__ __launch_bounds__(256) void k_slices_begin(const float4* __restrict__ rec, float4* __restrict__ to,
                                                      float* __restrict__ ds, int64_t n_dst, int H)
{
    const int64_t total = n_dst * H;
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < total; x += (int64_t)gridDim.x * 256) {
        const int64_t i = x / H;
        const int h = (int)(x - i * H);
        to[((h / HS) * n_dst + i) * HS + h % HS] = rec[x];
        ds[x] = 0.f;
    }
}
template <int HS>
__global__ __launch_bounds__(256) void k_slices_end(const float* __restrict__ from, float* __restrict__ ds, int64_t n_dst,
                                                    int H)
{
    const int64_t total = n_dst * H;
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < total; x += (int64_t)gridDim.x * 256) {
        const int64_t i = x / H;
        const int h = (int)(x - i * H);
        ds[x] += from[((h / HS) * n_dst + i) * HS + h % HS];
    }
}

// da_l[set * width + f] += sum over the set's workgroups of partial[workgroup][f]
static __global__ __launch_bounds__(256) void k_slices_da(const float* __restrict__ partial, int n_wgs, int sets, int width,
                                                   float* __restrict__ da_l)
{
    __shared__ float red[256];
    const int set = blockIdx.x / width, f = blockIdx.x % width, parts = kXcds / sets;
    float s = 0.f;
    for (int w = threadIdx.x; w < n_wgs * parts; w += 256) {
        const int wg = w / parts * kXcds + w % parts * sets + set;
        s += partial[(int64_t)wg * width + f];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) da_l[blockIdx.x] += red[0];
}

template <int LPH, int HS>
__global__ __launch_bounds__(kThreads<true>) void k_gat_bwd_slices(f256::BwdTabs tabs, f256::BwdP a, SetP sp)
{
    using T = float;
    constexpr int B = kBatch, kLanes = LPH * HS, kSlots = kWave / kLanes, D = 4 * LPH;
    constexpr bool SYNC = true;
    static_assert(B <= LPH && kLanes <= kWave, "a batch must fit a head group");
    __shared__ float part[kWaves<SYNC>][kWave][4];
    __shared__ GlobalPtr<const T> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<T> s_dZ[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<float> s_dt[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ip[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_ix[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_rank[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_Z[threadIdx.x] = static_cast<const T*>(tabs.Z[threadIdx.x]);
        s_t[threadIdx.x] = tabs.t[threadIdx.x];
        s_dZ[threadIdx.x] = static_cast<T*>(tabs.dZ[threadIdx.x]);
        s_dt[threadIdx.x] = tabs.dt[threadIdx.x];
        s_ip[threadIdx.x] = tabs.t_indptr[threadIdx.x];
        s_ix[threadIdx.x] = tabs.t_indices[threadIdx.x];
        s_rank[threadIdx.x] = tabs.rank[threadIdx.x];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = lane / kLanes, hh = lane % kLanes / LPH, k = lane % LPH;
    const uint32_t mask = (1u << a.tag_shift) - 1u;
    const Unit<SYNC> u(a.H / HS);
    const int h = u.set * HS + hh, foff = h * D + 4 * k;
    const T* Gp = static_cast<const T*>(a.G) + foff;
    const float4* rec_of = sp.rec + (int64_t)u.set * sp.n_dst * HS + hh;
    float* ds_of = sp.ds + (int64_t)u.set * sp.n_dst * HS + hh;
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4] = {0.f, 0.f, 0.f, 0.f};
    load_f32<4>(a.a_l + foff, al);
    int64_t r0 = u.first(wave, kSlots);
    for (int64_t w0 = SYNC ? u.first(0, kSlots) : r0; w0 < a.n_rows; w0 += u.stride(kSlots), r0 += u.stride(kSlots)) {
        const bool live = r0 + slot < a.n_rows;
        const uint32_t id = a.rows[live ? r0 + slot : a.n_rows - 1];
        const int q = (int)(id >> a.tag_shift), j = (int)(id & mask);
        const int32_t* idx = s_ix[q];
        const int beg = s_ip[q][j], len = s_ip[q][j + 1] - beg;      // (at least 8)
        float zj[4];
        Row4<T>::unpack(load_lane<T, false>(s_Z[q] + (int64_t)j * a.ld, foff, true), zj);
        float t2;
        if (s_t[q]) {
            t2 = f256::score_log2(s_t[q][(int64_t)j * a.ldh + h]);
        } else {
            float c = al[0] * zj[0];
#pragma unroll
            for (int x = 1; x < 4; ++x) c = fmaf(al[x], zj[x], c);
            t2 = f256::score_log2(group_all<LPH, OpSum>(c));
        }
        float dz[4] = {0.f, 0.f, 0.f, 0.f}, dt = 0.f;
        int mine = idx[beg + min(k, len - 1)];
        for (int e0 = 0, turn = 0; go_on<SYNC>(e0 < len, turn); e0 += B, ++turn) {
            if (e0 >= len) continue;
            const int next = idx[beg + min(e0 + B + k, len - 1)];
            typename Row4<T>::Raw raw[B];
            const Spread<LPH, LPH <= 32> ids(mine);
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                raw[K] = load_lane<T, false>(Gp + (uint64_t)(uint32_t)ids.template of_int<K>() * (uint32_t)a.ld, 0, true);
            });
            const float4 rec = rec_of[(int64_t)mine * HS];
            loads_sent();
            zero_behind(raw, len - e0);
            const bool valid = live && k < B && e0 + k < len;
            float c_mine = 0.f;
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                float g[4];
                Row4<T>::unpack(raw[K], g);
                float c = g[0] * zj[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(g[x], zj[x], c);
                c = group_all<LPH, OpSum>(c);
                c_mine = k == K ? c : c_mine;
            });
            const float u2 = rec.x + t2;
            const float alpha = f256::alpha_if(valid, u2, a.slope, rec.y);
            const float de = alpha * (c_mine - rec.z);
            const float du = u2 > 0.f ? de : a.slope * de;
            dt += valid ? du : 0.f;
            if (valid) unsafeAtomicAdd(ds_of + (int64_t)mine * HS, du);
            const Spread<LPH, LPH <= 32> as(alpha);
            static_for<B>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float ak = as.template of<K>();
                float g[4];
                Row4<T>::unpack(raw[K], g);
#pragma unroll
                for (int x = 0; x < 4; ++x) dz[x] = fmaf(ak, g[x], dz[x]);
            });
            mine = next;
        }
        // dZ_q[j] = sum alpha G + dt a_l ; dt_q[j] = dt ; da_l += dt z_j
        dt = group_all<LPH, OpSum>(dt);
        if (live) {
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] = fmaf(dt, al[x], dz[x]);
                dal[x] = fmaf(dt, zj[x], dal[x]);
            }
            const int64_t jo = s_rank[q] ? s_rank[q][j] : j;
            store_lane<T, false>(s_dZ[q] + jo * a.ld, foff, true, v);
            if (k == 0 && s_dt[q]) s_dt[q][jo * a.ldh + h] = dt;
        }
    }
    // this workgroup's share of the set's da_l
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) part[wave][lane][x] = dal[x];
    __syncthreads();
    constexpr int width = HS * D;
    if ((int)threadIdx.x < width) {
        const int f = (int)threadIdx.x, from = f / D * LPH + f % D / 4, x = f % 4;
        float s = 0.f;
        for (int w = 0; w < kWaves<SYNC>; ++w)
#pragma unroll
            for (int y = 0; y < kSlots; ++y) s += part[w][y * kLanes + from][x];
        a.partial[(int64_t)blockIdx.x * width + f] = s;
    }
}

}  // namespace slices

// The forward pass over all blocks (sync: the table does not fit in L2; heads of 128 bytes to 128 values) and the fp32
// backward pass over the sources of 8 edges and more (rows, n_rows; heads of 32, 64 or 128 values, whole sets; records and
// ds of every destination and head in the caller's scratch), all heads at once; parameters as for gat_f256.h.
int fwd_slices(int dtype, const f256::FwdP& p, const f256::Tabs& tabs, bool sync, hipStream_t st);
int bwd_slices(const f256::BwdP& p, const f256::BwdTabs& tabs, int64_t n_dst, void* scratch, float* ds, float* da_l,
               hipStream_t st);

inline int slice_lanes(int D) { return D <= 32 ? 8 : D <= 64 ? 16 : 32; }    // of a head

}  // namespace sar
