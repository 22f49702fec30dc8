// Attention kernels for layers whose heads leave room in a wavefront: narrow layers (one head of
// 47 values, 4 heads of 16, 4 of 32 ...) and layers whose head width is no multiple of 4.
//
// A head is covered by LPH lanes of 4 values (the power of two >= D/4), as in the padded geometry
// of gat_f256.h, and the 64/LPH lane groups of a wavefront that the heads do not need are not left
// idle: they form further SLOTS, group g speaking for head g % H of slot g / H.  In the forward
// kernel and in the backward kernel for sources of 8 and more edges the slots take different edges
// of the same row (each with its own running softmax, merged at the end of the row); in the
// backward kernel for the other sources every slot takes a source of its own.  A row of 188 bytes
// then costs a quarter of a wave-wide load instead of a whole one.
//
// Head widths that are no multiple of 4 (template flag RAG): the last lane of a head takes the LAST
// four values of the head instead of a piece that would end behind it, so every access is one
// (unaligned) 16- or 8-byte access inside the row.  The values it shares with the lane before it
// are left out of its dot products; where it accumulates or stores them it has the same bits as
// that lane.
//
// What bounds them: the bytes of the gathered rows (whole cache lines: a 188-byte row touches
// four 64-byte sectors), like the kernels of gat_f256.h; in the backward kernel of a small layer also the
// atomics on ds.  Measured on a worker's share of 7.4M edges, 1 x 47 fp32: kernels that moved one value
// per lane and reduced a head of 47 lanes by 47 shuffles per edge took 5.77 ms forward and 6.56 ms
// backward, these take 0.28 and 0.51 ms.
#pragma once

#include "gat_f256.h"

namespace sar {
namespace slots {

using f256::BwdAcc4;
using f256::BwdP;
using f256::alpha_if;
using f256::BwdTabs;
using f256::DsLater;
using f256::FwdP;
using f256::group_all;
using f256::leaky2;
using f256::OpMax;
using f256::OpSum;
using f256::Row4;
using f256::score_log2;
using f256::Spread;
using f256::static_for;
using f256::Tabs;

// Edges of one row (or of one source) a lane group has in flight.
template <int LPH>
constexpr int kBatch = LPH >= 8 ? 8 : 4;

// Where this lane stands.
template <int LPH, bool RAG>
struct Place {
    int lane, k_pos;   // lane of the wavefront, lane of the head group
    int slot, h;       // slot and head of the lane group
    bool live;         // the group has a slot (64/LPH need not be a multiple of H)
    bool on;           // the lane carries values
    int foff;          // first of the lane's 4 values inside the launch's row
    int dup;           // how many of them the lane before it carries as well (RAG only)
    __device__ inline Place(int H, int D, int n_slots)
    {
        lane = threadIdx.x & (kWave - 1);
        k_pos = lane % LPH;
        const int grp = lane / LPH;
        slot = grp / H;
        h = grp - slot * H;
        live = slot < n_slots;
        on = live && 4 * k_pos < D;
        const int off = RAG ? min(4 * k_pos, D - 4) : 4 * k_pos;
        dup = (RAG && on) ? 4 * k_pos - off : 0;
        foff = h * D + off;
    }
    // v without the values the lane before it carries as well
    __device__ inline void own_only(float (&v)[4]) const
    {
        if constexpr (RAG) {
#pragma unroll
            for (int x = 0; x < 3; ++x) v[x] = x >= dup ? v[x] : 0.f;
        }
    }
};

using f256::load_raw;
using f256::store4;
template <bool ANY>
__device__ inline void load4_f32(const float* p, float (&v)[4])
{
    Row4<float>::unpack(load_raw<float, ANY>(p), v);
}

// The places of a batch that some slot of the wavefront has an edge for, in three groups [0, G1), [G1, G2), [G2, END) that
// are skipped whole where none has.  Rows that end inside a batch are most of what these kernels see: of a batch of eight
// a row of 8 edges fills two places with four slots and four with two, a source of one edge fills one, and an empty place
// costs some fourteen instructions (its sum over the head, its weight's way back, its multiply-adds).  Without them, and
// with the registers that the shorter live ranges free (112 -> 89: five wavefronts per SIMD instead of four), backward
// kernels of 1 x 47 fp32 on 7.4M edges 541 -> 480 us, 4 x 32 on 75000 sources of 136 thousand edges 52 -> 47.
template <int B, int G1, int G2, int END>
struct Places {
    bool any, more, most;     // uniform: some slot has an edge in group 0, 1, 2
    template <int FROM, int TO, int R, typename F>
    static __device__ inline void run(F& f)
    {
        constexpr int lo = FROM > R * B ? FROM - R * B : 0, hi = TO < R * B + B ? TO - R * B : B;
        if constexpr (lo < hi)
            static_for<hi - lo>([&](auto k) { f(std::integral_constant<int, lo + decltype(k)::value>{}); });
    }
    // f(K) for the places R * B + K of round R
    template <int R, typename F>
    __device__ inline void each(F f) const
    {
        run<0, G1, R>(f);
        if (more) run<G1, G2, R>(f);
        if (most) run<G2, END, R>(f);
    }
};

// Rows of fewer than 8 edges, one per slot: the lists hold them by degree class (4 to 7 edges, 2 or 3, one, none), so the
// rows of a wavefront are of one class but at the borders.
template <int B>
using FewPlaces = Places<B, 1, 3, 7>;
template <int B>
__device__ inline FewPlaces<B> few_places(int cnt)
{
    return {__builtin_amdgcn_ballot_w64(cnt > 0) != 0, __builtin_amdgcn_ballot_w64(cnt > 1) != 0,
            __builtin_amdgcn_ballot_w64(cnt > 3) != 0};
}

// Batches of one row, `left` edges from the batch's first on, dealt to the slots in turn.
template <int B>
using RowPlaces = Places<B, 2, 4, 8>;
template <int B>
__device__ inline RowPlaces<B> row_places(int left, int n_slots)
{
    return {true, left > 2 * n_slots, left > 4 * n_slots};
}

__device__ inline uint64_t shfl64(uint64_t v, int from)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, from), hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), from);
    return (uint64_t)hi << 32 | lo;
}

// Adds the slots' values to slot 0 (n_slots a power of two; the other slots are left with junk).
__device__ inline float sum_slots(float v, int lane, int n_slots, int width)
{
    for (int o = n_slots >> 1; o > 0; o >>= 1) v += __shfl(v, lane + o * width);
    return v;
}

// ------------------------------------------------------------------ forward

struct State {
    float m2, l, acc[4];   // running maximum (log2 units), this lane's share of the denominator, numerator
};

template <typename T, int LPH, bool ALL, bool FLY, bool RAG>
__device__ inline void fwd_chunk(State& st, const FwdP& a, const GlobalPtr<const void>* s_Z, const GlobalPtr<const float>* s_t,
                                 uint32_t mine, int cnt, int n_slots, const Place<LPH, RAG>& p, float s2,
                                 const float (&al)[4])
{
    constexpr int B = kBatch<LPH>;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    // where the rows of the lanes' edges are, looked up for the whole chunk at once
    const uint64_t row = (ALL ? s_Z[mine >> a.tag_shift].bits : reinterpret_cast<uint64_t>(a.Z)) +
                         (uint64_t)(mine & mask) * (uint32_t)(a.ld * (int)sizeof(T));
    for (int k0 = 0; k0 < cnt; k0 += B * n_slots) {
        typename Row4<T>::Raw raw[B];
        uint64_t from[B];
        const RowPlaces<B> some = row_places<B>(cnt - k0, n_slots);
        some.template each<0>([&](auto kk) {
            constexpr int K = decltype(kk)::value;
            raw[K] = typename Row4<T>::Raw{};
            from[K] = shfl64(row, min(k0 + K * n_slots + p.slot, cnt - 1));
        });
        if (p.on) {
            some.template each<0>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                if (k0 + K * n_slots < cnt)           // uniform: some slot has an edge here
                    raw[K] = load_raw<T, RAG>(GlobalPtr<const T>::at(from[K]) + p.foff);
            });
        }
        loads_sent();
        // lane k of a head group speaks for the k-th edge of its slot
        const int my_e = k0 + p.k_pos * n_slots + p.slot;
        const bool valid = p.live && p.k_pos < B && my_e < cnt;
        float tv = 0.f;
        if constexpr (FLY) {
            some.template each<0>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                float v[4];
                Row4<T>::unpack(raw[K], v);
                p.own_only(v);          // not only a_l: 0 x inf would be NaN where the lane before has inf
                float c = al[0] * v[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(al[x], v[x], c);
                c = group_all<LPH, OpSum>(c);
                tv = (p.k_pos == K) ? c : tv;
            });
        } else {
            const uint32_t my = (uint32_t)__shfl((int)mine, valid ? my_e : 0);
            const float* tb = ALL ? s_t[my >> a.tag_shift].template as<const float>() : a.t;
            tv = tb[(int64_t)(my & mask) * a.ldh + p.h];
        }
        const float e2 = valid ? leaky2(fmaf(tv, kLog2e, s2), a.slope) : -INFINITY;
        const float cmax = group_all<LPH, OpMax>(e2);
        if (__builtin_amdgcn_ballot_w64(cmax > st.m2)) {
            const float mn = fmaxf(st.m2, cmax);
            const float c = fast_exp2(st.m2 - (mn == -INFINITY ? 0.f : mn));   // no edge yet: exp2(-inf) = 0
            st.l *= c;
#pragma unroll
            for (int x = 0; x < 4; ++x) st.acc[x] *= c;
            st.m2 = mn;
        }
        const float pe = fast_exp2(e2 - (st.m2 == -INFINITY ? 0.f : st.m2));   // 0 for the lanes without an edge
        st.l += pe;
        const Spread<LPH> ps(pe);
        some.template each<0>([&](auto kk) {
            constexpr int K = decltype(kk)::value;
            const float pk = ps.template of<K>();
            float v[4];
            Row4<T>::unpack(raw[K], v);
#pragma unroll
            for (int x = 0; x < 4; ++x) st.acc[x] = fmaf(pk, v[x], st.acc[x]);
        });
    }
}

__device__ inline void merge_into(State& st, float om, float ol, const float (&oacc)[4])
{
    const float mn = fmaxf(st.m2, om), ref = (mn == -INFINITY) ? 0.f : mn;
    const float ca = fast_exp2(st.m2 - ref), cb = fast_exp2(om - ref);
    st.l = st.l * ca + ol * cb;
#pragma unroll
    for (int x = 0; x < 4; ++x) st.acc[x] = st.acc[x] * ca + oacc[x] * cb;
    st.m2 = mn;
}

// The rows of the list, by workgroup `block` of `n_blocks`.
template <typename T, int LPH, bool ALL, bool FLY, bool RAG>
__device__ inline void fwd_rows(const FwdP& a, const Tabs& tabs, int n_slots, int block, int n_blocks)
{
    __shared__ float part[kWavesPerWG][kWave][6];
    __shared__ GlobalPtr<const void> s_Z[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> s_t[SAR_MAX_BLOCKS];
    if constexpr (ALL) {
        if (threadIdx.x < SAR_MAX_BLOCKS) {
            s_Z[threadIdx.x] = tabs.Z[threadIdx.x];
            s_t[threadIdx.x] = tabs.t[threadIdx.x];
        }
        __syncthreads();
    }
    const Place<LPH, RAG> p(a.H, a.D, n_slots);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int width = a.H * LPH;                       // lanes of a slot
    const bool first = p.slot == 0;
    T* outp = static_cast<T*>(a.out);
    float al[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FLY) {
        if (p.on) load4_f32<RAG>(a.a_l + p.foff, al);
        p.own_only(al);
    }
    auto init = [&](State& st, int i, bool carry) {
        st.m2 = -INFINITY;
        st.l = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) st.acc[x] = 0.f;
        if constexpr (!ALL) {
            if (carry && first) {   // the state carried from the blocks already aggregated enters through slot 0
                st.m2 = a.m[(int64_t)i * a.ldh + p.h] * kLog2e;
                st.l = (p.k_pos == 0) ? a.l[(int64_t)i * a.ldh + p.h] : 0.f;
                if (p.on) load4_f32<RAG>(a.acc + (int64_t)i * a.ld + p.foff, st.acc);
            }
        }
    };
    auto edges_at = [&](int at, int end) { return p.lane < end - at ? a.indices[at + p.lane] : 0u; };
    // `mine`: edges_at(beg, end); a chunk's edges are read while the one before it is folded
    auto edges = [&](State& st, int beg, int end, int step, uint32_t mine, float s2) {
        for (int cb = beg; cb < end; cb += step) {
            const uint32_t next = edges_at(cb + step, end);
            fwd_chunk<T, LPH, ALL, FLY, RAG>(st, a, s_Z, s_t, mine, min(kWave, end - cb), n_slots, p, s2, al);
            mine = next;
        }
        // one state per head out of the slots' states; the denominator becomes the group's total
        st.l = group_all<LPH, OpSum>(st.l);
        for (int o = n_slots >> 1; o > 0; o >>= 1) {
            const int from = p.lane + o * width;
            const float om = __shfl(st.m2, from), ol = __shfl(st.l, from);
            float oacc[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) oacc[x] = __shfl(st.acc[x], from);
            merge_into(st, om, ol, oacc);
        }
    };
    auto finish = [&](const State& st, int i) {
        if (!first || !p.live) return;
        const float l = st.l;
        if constexpr (ALL) {
            const float inv = l > 0.f ? 1.f / l : 0.f;
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] = st.acc[x] * inv;
                if (a.act == SAR_ACT_RELU) v[x] = fmaxf(v[x], 0.f);
            }
            if (p.on) store4<T, RAG>(outp + (int64_t)i * a.ld + p.foff, v);
            if (p.k_pos == 0) a.L[(int64_t)i * a.ldh + p.h] = l > 0.f ? (st.m2 + fast_log2(l)) * kLn2 : -INFINITY;
        } else {
            if (p.on) store4<float, RAG>(a.acc + (int64_t)i * a.ld + p.foff, st.acc);
            if (p.k_pos == 0) {
                a.m[(int64_t)i * a.ldh + p.h] = st.m2 * kLn2;
                a.l[(int64_t)i * a.ldh + p.h] = l;
            }
        }
    };

    // the long rows at the head of the list: the four wavefronts share the row
    for (int64_t r = block; r < a.n_long; r += n_blocks) {
        const int i = (int)a.rows[r];
        State st;
        init(st, i, wave == 0);
        int beg = a.indptr[i], end = a.indptr[i + 1];
        const float s = a.s[(int64_t)i * a.ldh + p.h];
        const int step = row_share(beg, end, wave, kWavesPerWG);
        edges(st, beg, end, step, edges_at(beg, end), s * kLog2e);
#pragma unroll
        for (int x = 0; x < 4; ++x) part[wave][p.lane][x] = st.acc[x];
        part[wave][p.lane][4] = st.m2;
        part[wave][p.lane][5] = st.l;
        __syncthreads();
        if (wave == 0) {
            for (int w = 1; w < kWavesPerWG; ++w) {
                float oacc[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) oacc[x] = part[w][p.lane][x];
                merge_into(st, part[w][p.lane][4], part[w][p.lane][5], oacc);
            }
            finish(st, i);
        }
        __syncthreads();
    }
    const int64_t n_waves = (int64_t)n_blocks * kWavesPerWG;
    // The other rows, 64 of a wavefront's at a time, as in f256::fwd_rows: lane u reads what there is to know of the u-th.
    // (With the addresses looked up by lanes, 38 layers: 8% shorter on average, 4 x 16 bf16 on 0.3 M rows of 26 320 -> 241 us.  The
    // wide backward kernel of the slots keeps a source's loads in line: the registers of this cost it a wavefront per SIMD.)
    for (int64_t r = a.n_long + from_behind(a.n_long, block, n_blocks) * kWavesPerWG + wave; r < a.n_rows;
         r += n_waves * kWave) {
        const bool have = r + p.lane * n_waves < a.n_rows;
        const int count = __builtin_popcountll(__builtin_amdgcn_ballot_w64(have));
        int row = 0, row_beg = 0, row_end = 0;
        if (have) {
            row = (int)a.rows[r + p.lane * n_waves];
            row_beg = a.indptr[row];
            row_end = a.indptr[row + 1];
        }
        auto of = [&](int v, int u) { return __builtin_amdgcn_readlane(v, u); };
        uint32_t mine = edges_at(of(row_beg, 0), of(row_end, 0));
        float s = a.s[(int64_t)of(row, 0) * a.ldh + p.h];
        for (int u = 0; u < count; ++u) {
            const int i = of(row, u), beg = of(row_beg, u), end = of(row_end, u), v = min(u + 1, count - 1);
            const uint32_t mine_next = edges_at(of(row_beg, v), of(row_end, v));
            const float s_next = a.s[(int64_t)of(row, v) * a.ldh + p.h];
            State st;
            init(st, i, true);
            edges(st, beg, end, kWave, mine, s * kLog2e);
            finish(st, i);
            mine = mine_next;
            s = s_next;
        }
    }
}

template <typename T, int LPH, bool FLY, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_gat_fwd_slots(FwdP a, Tabs tabs, int n_slots)
{
    fwd_rows<T, LPH, true, FLY, RAG>(a, tabs, n_slots, (int)blockIdx.x, (int)gridDim.x);
}

// Rows of fewer than 8 edges in the block of a per-block call: a P-way split leaves most rows two or three.  Every slot
// takes a row of its own, lane k of each of its head groups speaking for the row's edge k, so a row is one round of
// gathers (two of four where a head has only four lanes), and the carried state, read and written back, is most of what
// a row moves.  A wavefront for such a row alone waited for its list entry, its range, its edges and its sources in turn;
// here list entries are read three rounds ahead, ranges two, sources one.
template <typename T, int LPH, bool FLY, bool RAG>
__device__ inline void fwd_few(const FwdP& a, int n_slots, int64_t r_begin, int64_t r_end, int block, int n_blocks)
{
    constexpr int B = kBatch<LPH>;
    constexpr int kRounds = ((1 << kNarrowMaxClass) - 1 + B - 1) / B;
    const Place<LPH, RAG> p(a.H, a.D, n_slots);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T* Z = static_cast<const T*>(a.Z);
    float al[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FLY) {
        if (p.on) load4_f32<RAG>(a.a_l + p.foff, al);
        p.own_only(al);
    }
    struct Meta { int i, beg, cnt; };
    struct Src { int j[kRounds]; };
    const int64_t stride = (int64_t)n_blocks * kWavesPerWG * n_slots;
    const int64_t w0 = r_begin + ((int64_t)block * kWavesPerWG + wave) * n_slots;   // slot 0's list position
    auto have = [&](int64_t w) { return p.live && w + p.slot < r_end; };
    auto load_id = [&](int64_t w) { return have(w) ? (int)a.rows[w + p.slot] : 0; };
    auto load_meta = [&](int i, int64_t w) {
        Meta m{0, 0, 0};
        if (have(w)) {
            m.i = i;
            m.beg = a.indptr[i];
            m.cnt = a.indptr[i + 1] - m.beg;
        }
        return m;
    };
    auto load_src = [&](const Meta& m) {
        Src s;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int e = r * B + p.k_pos;
            s.j[r] = (p.k_pos < B && e < m.cnt) ? (int)a.indices[m.beg + e] : 0;
        }
        return s;
    };
    int id2 = load_id(w0 + 2 * stride);
    Meta m0 = load_meta(load_id(w0), w0), m1 = load_meta(load_id(w0 + stride), w0 + stride);
    Src s0 = load_src(m0);
    for (int64_t w = w0; w < r_end; w += stride) {
        const Src s1 = load_src(m1);
        const Meta m2 = load_meta(id2, w + 2 * stride);
        const int id3 = load_id(w + 3 * stride);
        const bool mine = have(w);
        const int64_t i = m0.i;
        State st{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
        float s2 = 0.f;
        const FewPlaces<B> some = few_places<B>(m0.cnt);
        if (mine) {
            if (p.on) load4_f32<RAG>(a.acc + i * a.ld + p.foff, st.acc);
            st.m2 = a.m[i * a.ldh + p.h] * kLog2e;
            st.l = p.k_pos == 0 ? a.l[i * a.ldh + p.h] : 0.f;
            s2 = a.s[i * a.ldh + p.h] * kLog2e;
        }
        static_for<kRounds>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            if (!(r == 0 ? some.any : some.most)) return;
            typename Row4<T>::Raw raw[B];
            const Spread<LPH> js(s0.j[r]);
            some.template each<r>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                raw[K] = typename Row4<T>::Raw{};
                const int j = js.template of_int<K>();
                if (p.on && r * B + K < m0.cnt) raw[K] = load_raw<T, RAG>(Z + (int64_t)j * a.ld + p.foff);
            });
            loads_sent();
            const bool valid = p.live && p.k_pos < B && r * B + p.k_pos < m0.cnt;
            float tv = 0.f;
            if constexpr (FLY) {
                some.template each<r>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    float v[4];
                    Row4<T>::unpack(raw[K], v);
                    p.own_only(v);
                    float c = al[0] * v[0];
#pragma unroll
                    for (int x = 1; x < 4; ++x) c = fmaf(al[x], v[x], c);
                    c = group_all<LPH, OpSum>(c);
                    tv = (p.k_pos == K) ? c : tv;
                });
            } else {
                if (valid) tv = a.t[(int64_t)s0.j[r] * a.ldh + p.h];
            }
            const float e2 = valid ? leaky2(fmaf(tv, kLog2e, s2), a.slope) : -INFINITY;
            const float mn = fmaxf(st.m2, group_all<LPH, OpMax>(e2)), ref = mn == -INFINITY ? 0.f : mn;
            const float c = fast_exp2(st.m2 - ref);      // no edge yet: 0
            const float pe = fast_exp2(e2 - ref);        // 0 for the lanes without an edge
            st.l = st.l * c + pe;
#pragma unroll
            for (int x = 0; x < 4; ++x) st.acc[x] *= c;
            st.m2 = mn;
            const Spread<LPH> ps(pe);
            some.template each<r>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float pk = ps.template of<K>();
                float v[4];
                Row4<T>::unpack(raw[K], v);
#pragma unroll
                for (int x = 0; x < 4; ++x) st.acc[x] = fmaf(pk, v[x], st.acc[x]);
            });
        });
        const float l = group_all<LPH, OpSum>(st.l);
        if (mine) {
            if (p.on) store4<float, RAG>(a.acc + i * a.ld + p.foff, st.acc);
            if (p.k_pos == 0) {
                a.m[i * a.ldh + p.h] = st.m2 * kLn2;
                a.l[i * a.ldh + p.h] = l;
            }
        }
        m0 = m1;
        s0 = s1;
        m1 = m2;
        id2 = id3;
    }
}

// A per-block call: the first n_wide workgroups take the rows of 8 edges and more (a.rows up to a.n_rows; WHOLE: by
// f256::fwd_rows, a wavefront's lanes on one edge of a row, otherwise by slots), the others [r_begin, r_end) of the list.
template <typename T, int LPH, bool FLY, bool RAG, bool WHOLE, bool PAD>
__global__ __launch_bounds__(kGatherThreads) void k_gat_fwd_block(FwdP a, int n_slots, int n_wide, int64_t r_begin,
                                                                  int64_t r_end)
{
    const Tabs none{};
    if ((int)blockIdx.x >= n_wide)
        fwd_few<T, LPH, FLY, RAG>(a, n_slots, r_begin, r_end, (int)blockIdx.x - n_wide, (int)gridDim.x - n_wide);
    else if constexpr (WHOLE)
        f256::fwd_rows<T, LPH, kBatch<LPH>, false, FLY, PAD>(a, none, (int)blockIdx.x, n_wide);
    else
        fwd_rows<T, LPH, false, FLY, RAG>(a, none, n_slots, (int)blockIdx.x, n_wide);
}

// ----------------------------------------------------------------- backward

// This workgroup's share of da_l = sum_j dt_j z_j, one row of 256 lane values per workgroup.
template <int LPH, bool RAG>
__device__ inline void store_partial(float (&dal)[4], float (*part)[kWave][4], const Place<LPH, RAG>& p, int wave,
                                     int n_slots, int width, float* row)
{
#pragma unroll
    for (int x = 0; x < 4; ++x) part[wave][p.lane][x] = sum_slots(dal[x], p.lane, n_slots, width);
    __syncthreads();
    if (wave == 0) {
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float s = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) s += part[w][p.lane][x];
            v[x] = s;
        }
        store_f32<4>(row + p.lane * 4, v);
    }
}

// Sources of at least 8 edges: one wavefront each (a workgroup for the long ones), its slots taking
// different edges.
template <typename T, int LPH, bool ALL, bool RAG>
__device__ inline void bwd_wide(const BwdTabs& tabs, const BwdP& a, int n_slots, int block, int n_blocks,
                                float* partial_row)
{
    constexpr int B = kBatch<LPH>;
    __shared__ float part[kWavesPerWG][kWave][4];
    __shared__ float part_dt[kWavesPerWG][kWave];
    const Place<LPH, RAG> p(a.H, a.D, n_slots);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int width = a.H * LPH;
    const bool first = p.slot == 0;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    const T* Gp = static_cast<const T*>(a.G);
    float* const ds = f256::ds_of(a);
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4];
    if (p.on) load4_f32<RAG>(a.a_l + p.foff, al);
#pragma unroll
    for (int x = 0; x < 4; ++x) dal[x] = 0.f;

    // (Heads of 16 lanes and more gain nothing by it and lose a wavefront per SIMD to its registers.)
    constexpr bool kLater = LPH <= 8;
    DsLater later;
    auto edges = [&](BwdAcc4& ac, int q, int j, int share, int shares, float (&zj)[4]) {
        typename Row4<T>::Raw zr{};
        if (p.on) zr = load_raw<T, RAG>(static_cast<const T*>(tabs.Z[q]) + (int64_t)j * a.ld + p.foff);
        Row4<T>::unpack(zr, zj);
        p.own_only(zj);
        float t2;
        if (tabs.t[q]) {
            t2 = score_log2(tabs.t[q][(int64_t)j * a.ldh + p.h]);
        } else {   // t_j = <a_l, z_j>
            float c = al[0] * zj[0];
#pragma unroll
            for (int x = 1; x < 4; ++x) c = fmaf(al[x], zj[x], c);
            t2 = score_log2(group_all<LPH, OpSum>(c));
        }
        const int32_t* idx = tabs.t_indices[q];
        int beg = tabs.t_indptr[q][j], end = tabs.t_indptr[q][j + 1];
        const int step = row_share(beg, end, share, shares);
#pragma unroll
        for (int x = 0; x < 4; ++x) ac.dz[x] = 0.f;
        ac.dt = 0.f;
        for (int cb = beg; cb < end; cb += step) {
            const int cnt = min(kWave, end - cb);
            const int mine = (p.lane < cnt) ? idx[cb + p.lane] : 0;
            for (int k0 = 0; k0 < cnt; k0 += B * n_slots) {
                typename Row4<T>::Raw raw[B];
                const RowPlaces<B> some = row_places<B>(cnt - k0, n_slots);
                int e0 = k0 + p.slot;
                asm("" : "+v"(e0));
                some.template each<0>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    raw[K] = typename Row4<T>::Raw{};
                    if (k0 + K * n_slots < cnt) {
                        const int i = __shfl(mine, min(e0 + K * n_slots, cnt - 1));
                        if (p.on) raw[K] = load_raw<T, RAG>(Gp + (int64_t)i * a.ld + p.foff);
                    }
                });
                const int my_e = e0 + p.k_pos * n_slots;
                const bool valid = p.live && p.k_pos < B && my_e < cnt;
                const int my_i = __shfl(mine, valid ? my_e : 0);
                const float4 rec = a.rec[(int64_t)my_i * a.ldh + p.h];
                if constexpr (kLater) later.send();
                float c_mine = 0.f;
                some.template each<0>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    float g[4];
                    Row4<T>::unpack(raw[K], g);
                    float c = g[0] * zj[0];
#pragma unroll
                    for (int x = 1; x < 4; ++x) c = fmaf(g[x], zj[x], c);
                    c = group_all<LPH, OpSum>(c);
                    c_mine = (p.k_pos == K) ? c : c_mine;
                });
                const float u2 = rec.x + t2;
                const float alpha = alpha_if(valid, u2, a.slope, rec.y);
                const float de = alpha * (c_mine - rec.z);
                const float du = u2 > 0.f ? de : a.slope * de;
                ac.dt += du;
                later.set(valid, ds + (int64_t)my_i * a.ldh + p.h, du);
                if constexpr (!kLater) later.send();
                const Spread<LPH> as(alpha);
                some.template each<0>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const float ak = as.template of<K>();
                    float g[4];
                    Row4<T>::unpack(raw[K], g);
#pragma unroll
                    for (int x = 0; x < 4; ++x) ac.dz[x] = fmaf(ak, g[x], ac.dz[x]);
                });
            }
        }
        ac.dt = sum_slots(group_all<LPH, OpSum>(ac.dt), p.lane, n_slots, width);
#pragma unroll
        for (int x = 0; x < 4; ++x) ac.dz[x] = sum_slots(ac.dz[x], p.lane, n_slots, width);
    };
    // dZ_q[j] = sum alpha G + dt a_l ; dt_q[j] = dt ; da_l += dt z_j (slot 0 holds the sums)
    auto outputs = [&](const BwdAcc4& ac, int q, int j, const float (&zj)[4]) {
        if (!first || !p.live) return;
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            v[x] = fmaf(ac.dt, al[x], ac.dz[x]);
            dal[x] = fmaf(ac.dt, zj[x], dal[x]);
        }
        const int64_t jo = tabs.rank[q] ? tabs.rank[q][j] : j;
        if (p.on) store4<T, RAG>(static_cast<T*>(tabs.dZ[q]) + jo * a.ld + p.foff, v);
        if (p.k_pos == 0 && tabs.dt[q]) tabs.dt[q][jo * a.ldh + p.h] = ac.dt;
    };

    for (int64_t r = block; r < a.n_long; r += n_blocks) {
        const uint32_t id = a.rows[r];
        const int q = ALL ? (int)(id >> a.tag_shift) : 0, j = (int)(id & mask);
        BwdAcc4 ac;
        float zj[4];
        edges(ac, q, j, wave, kWavesPerWG, zj);
#pragma unroll
        for (int x = 0; x < 4; ++x) part[wave][p.lane][x] = ac.dz[x];
        part_dt[wave][p.lane] = ac.dt;
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                float s = 0.f;
                for (int w = 0; w < kWavesPerWG; ++w) s += part[w][p.lane][x];
                ac.dz[x] = s;
            }
            float s = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) s += part_dt[w][p.lane];
            ac.dt = s;
            outputs(ac, q, j, zj);
        }
        __syncthreads();
    }
    const int64_t n_waves = (int64_t)n_blocks * kWavesPerWG;
    for (int64_t r = a.n_long + from_behind(a.n_long, block, n_blocks) * kWavesPerWG + wave; r < a.n_rows; r += n_waves) {
        const uint32_t id = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.rows[r]);
        const int q = ALL ? (int)(id >> a.tag_shift) : 0, j = (int)(id & mask);
        BwdAcc4 ac;
        float zj[4];
        edges(ac, q, j, 0, 1, zj);
        outputs(ac, q, j, zj);
    }
    later.send();
    __syncthreads();
    store_partial<LPH, RAG>(dal, part, p, wave, n_slots, width, partial_row);
}

// The other sources of the list (fewer than 8 edges, or none): every slot takes a source of its
// own, lane k of each of its head groups speaking for the source's edge k, so a source is one
// round of gathers (two of four where a head has only four lanes).  List entries are read three
// rounds ahead, ranges and output rows two, destinations one.
template <typename T, int LPH, bool ALL, bool RAG>
__device__ inline void bwd_few(const BwdTabs& tabs, const BwdP& a, int n_slots, int64_t r_begin, int64_t r_end,
                               int block, int n_blocks, float* partial_row)
{
    constexpr int B = kBatch<LPH>;
    constexpr int kMost = 1 << kNarrowMaxClass;          // this kernel's sources have fewer edges
    constexpr int kRounds = (kMost - 1 + B - 1) / B;
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
    const Place<LPH, RAG> p(a.H, a.D, n_slots);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int width = a.H * LPH;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    const T* Gp = static_cast<const T*>(a.G);
    float* const ds = f256::ds_of(a);
    float al[4] = {0.f, 0.f, 0.f, 0.f}, dal[4];
    if (p.on) load4_f32<RAG>(a.a_l + p.foff, al);
#pragma unroll
    for (int x = 0; x < 4; ++x) dal[x] = 0.f;

    struct Meta { int q, j, beg, cnt, jo; };
    struct Dst { int i[kRounds]; };
    const int64_t stride = (int64_t)n_blocks * kWavesPerWG * n_slots;
    const int64_t w0 = r_begin + ((int64_t)block * kWavesPerWG + wave) * n_slots;   // slot 0's list position
    auto have = [&](int64_t w) { return p.live && w + p.slot < r_end; };
    auto load_id = [&](int64_t w) -> uint32_t { return have(w) ? a.rows[w + p.slot] : 0u; };
    auto load_meta = [&](uint32_t id, int64_t w) {
        Meta m{0, 0, 0, 0, 0};
        if (have(w)) {
            m.q = ALL ? (int)(id >> a.tag_shift) : 0;
            m.j = (int)(id & mask);
            const int32_t* ip = s_ip[m.q];
            m.beg = ip[m.j];
            m.cnt = ip[m.j + 1] - m.beg;
            m.jo = s_rank[m.q] ? s_rank[m.q][m.j] : m.j;
        }
        return m;
    };
    auto load_dst = [&](const Meta& m) {
        Dst d;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int e = r * B + p.k_pos;
            d.i[r] = (p.k_pos < B && e < m.cnt) ? s_ix[m.q][m.beg + e] : 0;
        }
        return d;
    };
    uint32_t id2 = load_id(w0 + 2 * stride);
    Meta m0 = load_meta(load_id(w0), w0), m1 = load_meta(load_id(w0 + stride), w0 + stride);
    Dst d0 = load_dst(m0);

    for (int64_t w = w0; w < r_end; w += stride) {
        const Dst d1 = load_dst(m1);
        const Meta m2 = load_meta(id2, w + 2 * stride);
        const uint32_t id3 = load_id(w + 3 * stride);
        const bool mine = have(w);
        const FewPlaces<B> some = few_places<B>(m0.cnt);
        float zj[4];
        {
            typename Row4<T>::Raw zr{};
            if (m0.cnt > 0 && p.on) zr = load_raw<T, RAG>(s_Z[m0.q].template as<const T>() + (int64_t)m0.j * a.ld + p.foff);
            Row4<T>::unpack(zr, zj);
            p.own_only(zj);
        }
        float dz[4] = {0.f, 0.f, 0.f, 0.f}, dt = 0.f, t2 = 0.f;
        static_for<kRounds>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            if (!(r == 0 ? some.any : some.most)) return;
            typename Row4<T>::Raw raw[B];
            const Spread<LPH> is(d0.i[r]);
            some.template each<r>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                raw[K] = typename Row4<T>::Raw{};
                const int i = is.template of_int<K>();
                if (p.on && r * B + K < m0.cnt) raw[K] = load_raw<T, RAG>(Gp + (int64_t)i * a.ld + p.foff);
            });
            const bool valid = p.live && p.k_pos < B && r * B + p.k_pos < m0.cnt;
            const int my_i = d0.i[r];
            float4 rec = make_float4(0.f, INFINITY, 0.f, 0.f);   // L = +inf gives alpha = 0
            if (valid) rec = a.rec[(int64_t)my_i * a.ldh + p.h];
            loads_sent();
            if constexpr (r == 0) {
                float c = al[0] * zj[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(al[x], zj[x], c);
                c = group_all<LPH, OpSum>(c);
                if (mine && s_t[m0.q]) c = s_t[m0.q][(int64_t)m0.j * a.ldh + p.h];
                t2 = score_log2(c);
            }
            float c_mine = 0.f;
            some.template each<r>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                float g[4];
                Row4<T>::unpack(raw[K], g);
                float c = g[0] * zj[0];
#pragma unroll
                for (int x = 1; x < 4; ++x) c = fmaf(g[x], zj[x], c);
                c = group_all<LPH, OpSum>(c);
                c_mine = (p.k_pos == K) ? c : c_mine;
            });
            const float u2 = rec.x + t2;
            const float alpha = alpha_if(valid, u2, a.slope, rec.y);
            const float de = alpha * (c_mine - rec.z);
            const float du = u2 > 0.f ? de : a.slope * de;
            dt += du;
            if (valid) unsafeAtomicAdd(ds + (int64_t)my_i * a.ldh + p.h, du);
            const Spread<LPH> as(alpha);
            some.template each<r>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float ak = as.template of<K>();
                float g[4];
                Row4<T>::unpack(raw[K], g);
#pragma unroll
                for (int x = 0; x < 4; ++x) dz[x] = fmaf(ak, g[x], dz[x]);
            });
        });
        dt = group_all<LPH, OpSum>(dt);
        if (mine) {
            float v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] = fmaf(dt, al[x], dz[x]);
                dal[x] = fmaf(dt, zj[x], dal[x]);
            }
            if (p.on) store4<T, RAG>(s_dZ[m0.q].template as<T>() + (int64_t)m0.jo * a.ld + p.foff, v);
            if (p.k_pos == 0 && s_dt[m0.q]) s_dt[m0.q][(int64_t)m0.jo * a.ldh + p.h] = dt;
        }
        m0 = m1;
        d0 = d1;
        m1 = m2;
        id2 = id3;
    }
    store_partial<LPH, RAG>(dal, part, p, wave, n_slots, width, partial_row);
}

// One launch for both kinds of sources: the first n_wide workgroups share the wide ones (a.rows up to
// a.n_rows, the long ones first), the others [r_begin, r_end) of the list.  They do not depend on each other,
// and in a small call neither fills the chip: one after the other, the second waited for the first one's
// longest row, and a launch costs as much as some of them take (4 heads x 16 over 4096 nodes: 23.4 + 5.6 -> 24.0
// us; 16 blocks of 4 x 32, 75000 sources each: 37.4 + 31.1 -> 52.3 us a block).  Workgroup w leaves its part of da_l in
// row partial_row0 + w.
template <typename T, int LPH, bool ALL, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd_slots(BwdTabs tabs, BwdP a, int n_slots, int n_wide,
                                                                  int64_t r_begin, int64_t r_end, int partial_row0)
{
    float* const partial_row = a.partial + ((int64_t)partial_row0 + blockIdx.x) * f256::kF;
    const int b = blockIdx.x;
    if (b < n_wide)
        bwd_wide<T, LPH, ALL, RAG>(tabs, a, n_slots, b, n_wide, partial_row);
    else
        bwd_few<T, LPH, ALL, RAG>(tabs, a, n_slots, r_begin, r_end, b - n_wide, (int)gridDim.x - n_wide, partial_row);
}

}  // namespace slots
}  // namespace sar
