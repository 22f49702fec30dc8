// Sum / mean aggregation of neighbour features over partition blocks
// (Eq. 2 and the accumulation loop of Alg. 1), and its case-1 backward
// (Sec. 3.2: the gradient of a sum needs no features).
//
// All kernels are row gathers bound by HBM/L2 bandwidth: one wavefront owns one
// output row, reads the listed input rows with 16-byte lane accesses (a 1 KiB
// row is one wave-wide load), keeps several of them in flight, and adds them
// in fp32 registers.  The long rows at the head of a list are shared by the four
// wavefronts of a workgroup and merged through LDS.  The grid is persistent:
// workgroups stride over the degree-ordered row list, longest rows first.
//
// Rows of fewer than 512 bytes leave room for several lane groups in a wavefront: they take
// different edges of a row, or, for rows of fewer than 8 edges, a row each (k_rows_few).  Row widths
// that are no whole number of 16-byte pieces (template flag RAG): the last lane of a row takes the
// row's last 16 bytes, so every access is one unaligned 16-byte access inside the row; the values
// it shares with the lane before it get the same bits from both (and where sums are added to an
// accumulator that lane adds them alone).  A worker's 6.2M edges of bf16 rows of 47 values: forward 171 us,
// backward 142 us for the sources of 8 and more edges and 81 us for the others; the whole layer took 1.83 ms when
// such rows were moved 2 bytes per lane, 0.56 ms now.
#include <algorithm>

#include "gather_common.h"
#include "sar_internal.h"

namespace {

using namespace sar;

constexpr int kU = 4;   // rows in flight per lane group, twice as many where a row has them

struct PtrTab {
    const void* p[SAR_MAX_BLOCKS];
};

struct SpmmArgs {
    const int32_t* indptr;    // row offsets ([n+1]); per-block, all-blocks or transposed
    const uint32_t* indices;  // column ids (tagged with the block in the all-blocks index)
    const uint32_t* rows;     // launch list, longest class first
    int64_t n_rows, n_long;
    const void* Z;            // single input (per-block calls)
    float* acc;               // fp32 accumulator rows, read-modify-write (forward per block)
    void* out;                // typed output rows (batched forward, backward)
    const int32_t* deg;       // |N(i)| for the mean, or null
    int F;                    // values per row handled by this launch
    int ld;                   // stride between rows (values)
    int tag_shift;            // all-blocks index: block = id >> tag_shift
    int mean;
    const void* res;          // batched forward: rows added to the aggregate (Eq. 2's W_res h), or null
    int act;                  //                  SAR_ACT_* applied after that
    const int32_t* out_rank;  // backward, compact errors: row of `out` that source j owns (null: j)
};

enum class Mode { kBlock, kAll, kBackward };

// The lane's place in a row: the first of its VEC values and whether it carries any.
template <typename T, int G, bool RAG>
struct RowLanes {
    static constexpr int VEC = Vec<T>::N;
    int lane, gl, slot, off;
    bool on;
    __device__ inline explicit RowLanes(int F)
    {
        lane = threadIdx.x & (kWave - 1);
        gl = lane & (G - 1);
        slot = lane / G;
        on = gl * VEC < F;
        off = RAG ? min(gl * VEC, F - VEC) : gl * VEC;
    }
    static __device__ inline typename Vec<T>::Raw load(const T* p)
    {
        if constexpr (RAG) {
            typename Vec<T>::Raw r;
            __builtin_memcpy(&r, p, sizeof(r));
            return r;
        } else {
            return Vec<T>::load(p);
        }
    }
    static __device__ inline void store(T* p, const float (&v)[VEC])
    {
        if constexpr (RAG) {
            alignas(16) T tmp[VEC];
            Vec<T>::store(tmp, v);
            __builtin_memcpy(p, tmp, sizeof(tmp));
        } else {
            Vec<T>::store(p, v);
        }
    }
    // p[x] += v[x], p being this lane's place in an fp32 row.  The last lane of a ragged row leaves out the values
    // it shares with the lane before it: whether that lane has stored them when this one loads is not fixed.
    __device__ inline void add_to(float* p, const float (&v)[VEC]) const
    {
        const int dup = RAG ? gl * VEC - off : 0;
        if (dup == 0) {
            float cur[VEC];
            if constexpr (RAG)
                __builtin_memcpy(cur, p, sizeof(cur));
            else
                load_f32<VEC>(p, cur);
#pragma unroll
            for (int x = 0; x < VEC; ++x) cur[x] += v[x];
            if constexpr (RAG)
                __builtin_memcpy(p, cur, sizeof(cur));
            else
                store_f32<VEC>(p, cur);
        } else {
#pragma unroll
            for (int x = 1; x < VEC; ++x)
                if (x >= dup) p[x] += v[x];
        }
    }
};

// Adds the rows of KU edges per lane group into acc: edges k0 + k SLOTS + slot of the chunk whose
// ids the lanes hold in `mine`.  FULL: all of them are below cnt.
template <typename T, int G, Mode M, bool RAG, int KU, bool FULL>
__device__ inline void add_batch(float (&acc)[Vec<T>::N], const SpmmArgs& a, const GlobalPtr<const void>* ztab, uint32_t mine,
                                 int k0, int cnt, const RowLanes<T, G, RAG>& lm)
{
    constexpr int VEC = Vec<T>::N;
    constexpr int SLOTS = kWave / G;
    const uint32_t mask = (M == Mode::kAll) ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    typename Vec<T>::Raw raw[KU];
    int deg[KU];        // the weights are formed after all loads have been issued
#pragma unroll
    for (int k = 0; k < KU; ++k) {
        const int ek = k0 + k * SLOTS + lm.slot;
        const uint32_t id = __shfl(mine, ek & (kWave - 1));
        const bool ok = (FULL || ek < cnt) && lm.on;
        raw[k] = Vec<T>::zero();
        deg[k] = 1;
        if (ok) {
            const uint32_t j = id & mask;
            const T* base;
            if constexpr (M == Mode::kAll)
                base = ztab[id >> a.tag_shift].template as<const T>();
            else
                base = static_cast<const T*>(a.Z);
            raw[k] = lm.load(base + (int64_t)j * a.ld + lm.off);
            if constexpr (M == Mode::kBackward) {
                if (a.mean) deg[k] = a.deg[j];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < KU; ++k) {
        float v[VEC];
        Vec<T>::unpack(raw[k], v);
        const float w = 1.f / (float)max(deg[k], 1);
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            if constexpr (M == Mode::kBackward)
                acc[x] = fmaf(w, v[x], acc[x]);
            else
                acc[x] += v[x];
        }
    }
}

// Adds the rows listed in idx[beg,end) into acc; the wavefront takes share
// `share` of `shares` of them.  Eight edges per lane group are in flight while there are
// as many (forward, 7.4M edges: bf16 rows of 512 values 1208 us with four, 1099 with eight), then four.
// The backward pass over wide rows stays with four: a source has 12 edges on average and its wavefront
// waits for the chain in front of them, so what counts is how many wavefronts are resident (the same
// rows: 1149 us with four, 1257 with eight and their registers).
template <typename T, int G, Mode M, bool RAG>
__device__ inline void add_rows(float (&acc)[Vec<T>::N], const SpmmArgs& a, const GlobalPtr<const void>* ztab,
                                int beg, int end, int share, int shares, const RowLanes<T, G, RAG>& lm)
{
    constexpr int SLOTS = kWave / G;
    const int step = row_share(beg, end, share, shares);
    for (int cb = beg; cb < end; cb += step) {
        const int cnt = min(kWave, end - cb);
        const uint32_t mine = (lm.lane < cnt) ? a.indices[cb + lm.lane] : 0u;
        int k0 = 0;
        if constexpr (M != Mode::kBackward || G <= 16) {
            for (; k0 + 2 * kU * SLOTS <= cnt; k0 += 2 * kU * SLOTS)
                add_batch<T, G, M, RAG, 2 * kU, true>(acc, a, ztab, mine, k0, cnt, lm);
        }
        for (; k0 < cnt; k0 += kU * SLOTS) add_batch<T, G, M, RAG, kU, false>(acc, a, ztab, mine, k0, cnt, lm);
    }
}

template <typename T, int G>
__device__ inline void merge_slots(float (&acc)[Vec<T>::N])
{
#pragma unroll
    for (int o = G; o < kWave; o <<= 1)
#pragma unroll
        for (int x = 0; x < Vec<T>::N; ++x) acc[x] += __shfl_xor(acc[x], o);
}

template <typename T, int G, Mode M, bool RAG>
__device__ inline void finish_row(const float (&acc)[Vec<T>::N], const SpmmArgs& a, int i,
                                  const RowLanes<T, G, RAG>& lm)
{
    constexpr int VEC = Vec<T>::N;
    if (lm.slot != 0 || !lm.on) return;
    int64_t row = i;
    if constexpr (M == Mode::kBackward) {
        if (a.out_rank) row = a.out_rank[i];
    }
    const int64_t o = row * a.ld + lm.off;
    if constexpr (M == Mode::kBlock) {
        lm.add_to(a.acc + o, acc);
    } else {
        float v[VEC];
        float sc = 1.f;
        if constexpr (M == Mode::kAll) {
            if (a.mean) sc = 1.f / (float)max(a.deg[i], 1);
        }
#pragma unroll
        for (int x = 0; x < VEC; ++x) v[x] = acc[x] * sc;
        if constexpr (M == Mode::kAll) {
            if (a.res) {
                float r[VEC];
                Vec<T>::unpack(lm.load(static_cast<const T*>(a.res) + o), r);
#pragma unroll
                for (int x = 0; x < VEC; ++x) v[x] += r[x];
            }
            if (a.act == SAR_ACT_RELU) {
#pragma unroll
                for (int x = 0; x < VEC; ++x) v[x] = fmaxf(v[x], 0.f);
            }
        }
        lm.store(static_cast<T*>(a.out) + o, v);
    }
}

template <typename T, int G, Mode M, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_spmm(SpmmArgs a, PtrTab tab, int P)
{
    constexpr int VEC = Vec<T>::N;
    __shared__ GlobalPtr<const void> ztab[SAR_MAX_BLOCKS];
    __shared__ float part[kWavesPerWG][G][VEC];
    if constexpr (M == Mode::kAll) {
        if ((int)threadIdx.x < P) ztab[threadIdx.x] = tab.p[threadIdx.x];
        __syncthreads();
    }
    const RowLanes<T, G, RAG> lm(a.F);
    const int wave = threadIdx.x / kWave;

    // long rows: one workgroup each
    for (int64_t r = blockIdx.x; r < a.n_long; r += gridDim.x) {
        const int i = (int)a.rows[r];
        float acc[VEC] = {};
        add_rows<T, G, M, RAG>(acc, a, ztab, a.indptr[i], a.indptr[i + 1], wave, kWavesPerWG, lm);
        merge_slots<T, G>(acc);
        if (lm.slot == 0)
#pragma unroll
            for (int x = 0; x < VEC; ++x) part[wave][lm.gl][x] = acc[x];
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int x = 0; x < VEC; ++x) {
                float t = 0.f;
                for (int w = 0; w < kWavesPerWG; ++w) t += part[w][lm.gl][x];
                acc[x] = t;
            }
            finish_row<T, G, M, RAG>(acc, a, i, lm);
        }
        __syncthreads();
    }
    // remaining rows: one wavefront each
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t r = a.n_long + from_behind(a.n_long, blockIdx.x, gridDim.x) * kWavesPerWG + wave; r < a.n_rows; r += n_waves) {
        const int i = (int)a.rows[r];
        float acc[VEC] = {};
        add_rows<T, G, M, RAG>(acc, a, ztab, a.indptr[i], a.indptr[i + 1], 0, 1, lm);
        merge_slots<T, G>(acc);
        finish_row<T, G, M, RAG>(acc, a, i, lm);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_spmm_end(const int32_t* __restrict__ deg, int mean,
                                                  const float* __restrict__ acc, const T* res, int act, T* out,
                                                  int64_t n, int F)
{
    constexpr int VEC = Vec<T>::N;
    const int64_t total = n * (F / VEC);
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < total; k += (int64_t)gridDim.x * 256) {
        const int64_t i = k / (F / VEC);
        float v[VEC];
        load_f32<VEC>(acc + k * VEC, v);
        float sc = 1.f;
        if (mean) {
            const int d = deg[i];
            sc = d > 0 ? 1.f / (float)d : 0.f;
        }
#pragma unroll
        for (int x = 0; x < VEC; ++x) v[x] *= sc;
        if (res) {
            float r[VEC];
            Vec<T>::unpack(Vec<T>::load(res + k * VEC), r);
#pragma unroll
            for (int x = 0; x < VEC; ++x) v[x] += r[x];
        }
        if (act == SAR_ACT_RELU) {
#pragma unroll
            for (int x = 0; x < VEC; ++x) v[x] = fmaxf(v[x], 0.f);
        }
        Vec<T>::store(out + k * VEC, v);
    }
}

// G = dH * act'(.) with the derivative expressed through the output h (ReLU: 1 where h > 0)
template <typename T>
__global__ __launch_bounds__(256) void k_act_bwd(const T* h, const T* dH, T* G, int64_t n_vec)
{
    constexpr int VEC = Vec<T>::N;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n_vec; k += (int64_t)gridDim.x * 256) {
        float hv[VEC], g[VEC];
        Vec<T>::unpack(Vec<T>::load(h + k * VEC), hv);
        Vec<T>::unpack(Vec<T>::load(dH + k * VEC), g);
#pragma unroll
        for (int x = 0; x < VEC; ++x) g[x] = hv[x] > 0.f ? g[x] : 0.f;
        Vec<T>::store(G + k * VEC, g);
    }
}

// Case-1 backward over the sources of ALL blocks in one launch.  The work list holds
// (block << tag_shift) | source for every source of every block, longest first and
// the sources without an edge last (they get dZ = 0); each entry is one row of one
// block's transposed index.
struct BwdAllTabs {
    const int32_t* t_indptr[SAR_MAX_BLOCKS];
    const uint32_t* t_indices[SAR_MAX_BLOCKS];
    void* dZ[SAR_MAX_BLOCKS];
    const int32_t* rank[SAR_MAX_BLOCKS];
};

template <typename T, int G, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_spmm_bwd_all(SpmmArgs a, BwdAllTabs tabs)
{
    constexpr int VEC = Vec<T>::N;
    constexpr Mode M = Mode::kBackward;
    __shared__ float part[kWavesPerWG][G][VEC];
    const RowLanes<T, G, RAG> lm(a.F);
    const int wave = threadIdx.x / kWave;
    const uint32_t mask = (1u << a.tag_shift) - 1u;
    auto locate = [&](int64_t r, SpmmArgs& la) -> int {
        const uint32_t id = __builtin_amdgcn_readfirstlane(a.rows[r]);
        const uint32_t q = id >> a.tag_shift;
        la.indptr = tabs.t_indptr[q];
        la.indices = tabs.t_indices[q];
        la.out = tabs.dZ[q];
        la.out_rank = tabs.rank[q];
        return (int)(id & mask);
    };

    for (int64_t r = blockIdx.x; r < a.n_long; r += gridDim.x) {
        SpmmArgs la = a;
        const int j = locate(r, la);
        float acc[VEC] = {};
        add_rows<T, G, M, RAG>(acc, la, nullptr, la.indptr[j], la.indptr[j + 1], wave, kWavesPerWG, lm);
        merge_slots<T, G>(acc);
        if (lm.slot == 0)
#pragma unroll
            for (int x = 0; x < VEC; ++x) part[wave][lm.gl][x] = acc[x];
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int x = 0; x < VEC; ++x) {
                float t = 0.f;
                for (int w = 0; w < kWavesPerWG; ++w) t += part[w][lm.gl][x];
                acc[x] = t;
            }
            finish_row<T, G, M, RAG>(acc, la, j, lm);
        }
        __syncthreads();
    }
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t r = a.n_long + from_behind(a.n_long, blockIdx.x, gridDim.x) * kWavesPerWG + wave; r < a.n_rows; r += n_waves) {
        SpmmArgs la = a;
        const int j = locate(r, la);
        float acc[VEC] = {};
        add_rows<T, G, M, RAG>(acc, la, nullptr, la.indptr[j], la.indptr[j + 1], 0, 1, lm);
        merge_slots<T, G>(acc);
        finish_row<T, G, M, RAG>(acc, la, j, lm);
    }
}

// Rows of fewer than 8 edges and rows without any (list entries [r_begin, r_end)): a lane group
// each, all of a row's edges in flight at once.  One wavefront per such row left the memory system
// waiting for a chain of four dependent loads; list entries are read three rounds ahead here, ranges
// and output rows two, ids one.  ALLB: entries tagged with their block, as in k_spmm_bwd_all.
template <typename T, int G, Mode M, bool ALLB, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_rows_few(SpmmArgs a, BwdAllTabs tabs, int64_t r_begin, int64_t r_end)
{
    static_assert(M != Mode::kAll, "the all-blocks forward pass walks rows of all blocks together");
    constexpr int VEC = Vec<T>::N;
    constexpr int SLOTS = kWave / G;
    constexpr int kMost = (1 << sar::kNarrowMaxClass) - 1;
    constexpr int kHold = (kMost + G - 1) / G;          // ids a lane holds
    __shared__ GlobalPtr<const int32_t> s_ip[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const uint32_t> s_ix[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<void> s_out[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const int32_t> s_rank[SAR_MAX_BLOCKS];
    if constexpr (ALLB) {
        if (threadIdx.x < SAR_MAX_BLOCKS) {
            s_ip[threadIdx.x] = tabs.t_indptr[threadIdx.x];
            s_ix[threadIdx.x] = tabs.t_indices[threadIdx.x];
            s_out[threadIdx.x] = tabs.dZ[threadIdx.x];
            s_rank[threadIdx.x] = tabs.rank[threadIdx.x];
        }
        __syncthreads();
    }
    const RowLanes<T, G, RAG> lm(a.F);
    const uint32_t mask = ALLB ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    struct Meta { int q, j, beg, cnt, jo; };
    struct Ids { uint32_t v[kHold]; };
    const int64_t stride = (int64_t)gridDim.x * kWavesPerWG * SLOTS;
    const int64_t r0 = r_begin + ((int64_t)blockIdx.x * kWavesPerWG + threadIdx.x / kWave) * SLOTS + lm.slot;
    auto load_id = [&](int64_t r) -> uint32_t { return r < r_end ? a.rows[r] : 0u; };
    auto load_meta = [&](uint32_t id, int64_t r) {
        Meta m{0, 0, 0, 0, 0};
        if (r < r_end) {
            m.q = ALLB ? (int)(id >> a.tag_shift) : 0;
            m.j = (int)(id & mask);
            const int32_t* ip = ALLB ? s_ip[m.q].template as<const int32_t>() : a.indptr;
            m.beg = ip[m.j];
            m.cnt = ip[m.j + 1] - m.beg;
            m.jo = m.j;
            if constexpr (M == Mode::kBackward) {
                const int32_t* rank = ALLB ? s_rank[m.q].template as<const int32_t>() : a.out_rank;
                if (rank) m.jo = rank[m.j];
            }
        }
        return m;
    };
    auto load_ids = [&](const Meta& m) {
        Ids d;
#pragma unroll
        for (int k = 0; k < kHold; ++k) {
            const int e = k * G + lm.gl;
            d.v[k] = e < m.cnt ? (ALLB ? s_ix[m.q].template as<const uint32_t>() : a.indices)[m.beg + e] : 0u;
        }
        return d;
    };
    uint32_t id2 = load_id(r0 + 2 * stride);
    Meta m0 = load_meta(load_id(r0), r0), m1 = load_meta(load_id(r0 + stride), r0 + stride);
    Ids d0 = load_ids(m0);
    for (int64_t r = r0; r - lm.slot < r_end; r += stride) {       // uniform over the wavefront
        const Ids d1 = load_ids(m1);
        const Meta m2 = load_meta(id2, r + 2 * stride);
        const uint32_t id3 = load_id(r + 3 * stride);
        typename Vec<T>::Raw raw[kMost];
        int deg[kMost];
#pragma unroll
        for (int e = 0; e < kMost; ++e) {
            raw[e] = Vec<T>::zero();
            deg[e] = 1;
            const uint32_t j = __shfl(d0.v[e / G], lm.slot * G + e % G);
            if (e < m0.cnt && lm.on) {
                raw[e] = lm.load(static_cast<const T*>(a.Z) + (int64_t)j * a.ld + lm.off);
                if constexpr (M == Mode::kBackward) {
                    if (a.mean) deg[e] = a.deg[j];
                }
            }
        }
        if (r < r_end && lm.on) {
            float acc[VEC] = {};
#pragma unroll
            for (int e = 0; e < kMost; ++e) {
                float v[VEC];
                Vec<T>::unpack(raw[e], v);
                const float w = 1.f / (float)max(deg[e], 1);
#pragma unroll
                for (int x = 0; x < VEC; ++x) acc[x] = M == Mode::kBackward ? fmaf(w, v[x], acc[x]) : acc[x] + v[x];
            }
            const int64_t o = (int64_t)m0.jo * a.ld + lm.off;
            if constexpr (M == Mode::kBlock) {
                lm.add_to(a.acc + o, acc);
            } else {
                lm.store((ALLB ? s_out[m0.q].template as<T>() : static_cast<T*>(a.out)) + o, acc);
            }
        }
        m0 = m1;
        d0 = d1;
        m1 = m2;
        id2 = id3;
    }
}

// Ep[i] (+)= Eq[rank[i]] where source i of the block has a row in the compact error, else (+)= 0
template <typename T>
__global__ __launch_bounds__(256) void k_error_add(const T* __restrict__ Eq, const int32_t* __restrict__ rank,
                                                   int accumulate, T* Ep, int64_t n, int F)
{
    constexpr int VEC = Vec<T>::N;
    const int per_row = F / VEC;
    const int64_t total = n * per_row;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < total; k += (int64_t)gridDim.x * 256) {
        const int64_t i = k / per_row;
        const int c = (int)(k % per_row) * VEC;
        const int32_t r = rank[i];
        const bool has = rank[i + 1] > r;
        if (accumulate && !has) continue;
        float v[VEC];
#pragma unroll
        for (int x = 0; x < VEC; ++x) v[x] = 0.f;
        if (has) Vec<T>::unpack(Vec<T>::load(Eq + (int64_t)r * F + c), v);
        if (accumulate) {
            float e[VEC];
            Vec<T>::unpack(Vec<T>::load(Ep + i * F + c), e);
#pragma unroll
            for (int x = 0; x < VEC; ++x) v[x] += e[x];
        }
        Vec<T>::store(Ep + i * F + c, v);
    }
}

// Runs `...` with kG bound to the lanes of a row and kR to whether its accesses are the unaligned ones: the
// last lane is shifted back, or (a whole range of a row that is itself ragged) rows start anywhere.
#define SAR_DISPATCH_LANES(T, F, ld, ...)                                                      \
    do {                                                                                       \
        const bool ragged_ = (F) % Vec<T>::N != 0 || (ld) % Vec<T>::N != 0;                    \
        switch (lanes_for((F), Vec<T>::N)) {                                                   \
            case 4: { constexpr int kG = 4; SAR_RAGGED_OR_NOT(T, __VA_ARGS__); } break;         \
            case 8: { constexpr int kG = 8; SAR_RAGGED_OR_NOT(T, __VA_ARGS__); } break;         \
            case 16: { constexpr int kG = 16; SAR_RAGGED_OR_NOT(T, __VA_ARGS__); } break;       \
            case 32: { constexpr int kG = 32; SAR_RAGGED_OR_NOT(T, __VA_ARGS__); } break;       \
            default: { constexpr int kG = 64; SAR_RAGGED_OR_NOT(T, __VA_ARGS__); } break;       \
        }                                                                                      \
    } while (0)
#define SAR_RAGGED_OR_NOT(T, ...)                  \
    if (ragged_) {                                       \
        constexpr bool kR = Vec<T>::N * sizeof(T) == 16; \
        __VA_ARGS__;                               \
    } else {                                       \
        constexpr bool kR = false;                 \
        __VA_ARGS__;                               \
    }

// Rows of the list's tail with fewer than 8 edges go to k_rows_few where a wavefront has room for
// at least four of them (backward on 7.4M edges, alone -> with it: bf16 47 values 595 -> 318 us, fp32 64
// values 415 -> 371; with two to a wavefront it lost, fp32 128 values 603 -> 657).
template <typename T>
int64_t first_few(const SpmmArgs& a, int64_t n_wide)
{
    return lanes_for(a.F, Vec<T>::N) <= 16 ? std::min(n_wide, a.n_rows) : a.n_rows;
}
template <typename T>
unsigned few_grid(const SpmmArgs& a, int64_t n, int resident)
{
    const int64_t per_wg = (int64_t)kWavesPerWG * (kWave / lanes_for(a.F, Vec<T>::N));
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + per_wg - 1) / per_wg, resident));
}

// n_wide: list entries before it have at least 8 edges.
template <typename T, Mode M>
int launch_spmm(SpmmArgs a, const PtrTab& tab, int P, int64_t n_wide, hipStream_t st)
{
    if (a.n_rows == 0) return SAR_OK;
    if constexpr (M != Mode::kAll) {
        const int64_t few = first_few<T>(a, n_wide), n = a.n_rows - few;
        if (n > 0) {
            SAR_DISPATCH_LANES(T, a.F, a.ld, {
                auto fn = k_rows_few<T, (kG <= 16 ? kG : 16), M, false, kR>;
                static const int resident = resident_workgroups(fn);
                fn<<<few_grid<T>(a, n, resident), kGatherThreads, 0, st>>>(a, BwdAllTabs{}, few, a.n_rows);
            });
            SAR_LAUNCH_CHECK();
            a.n_rows = few;
            a.n_long = std::min(a.n_long, few);
            if (few == 0) return SAR_OK;
        }
    }
    // every workgroup of the persistent grid has to start at once: with 2048 of them and room for 1792,
    // the backward pass over rows of 512 bf16 values took 1580 us instead of 1149
    SAR_DISPATCH_LANES(T, a.F, a.ld, {
        auto fn = k_spmm<T, kG, M, kR>;
        static const int resident = resident_workgroups(fn);
        fn<<<persistent_grid_for(a.n_rows, a.n_long, resident), kGatherThreads, 0, st>>>(a, tab, P);
    });
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <typename T>
int launch_spmm_bwd_all(SpmmArgs a, const BwdAllTabs& tabs, int64_t n_wide, hipStream_t st)
{
    if (a.n_rows == 0) return SAR_OK;
    const int64_t few = first_few<T>(a, n_wide), n = a.n_rows - few;
    if (n > 0) {
        SAR_DISPATCH_LANES(T, a.F, a.ld, {
            auto fn = k_rows_few<T, (kG <= 16 ? kG : 16), Mode::kBackward, true, kR>;
            static const int resident = resident_workgroups(fn);
            fn<<<few_grid<T>(a, n, resident), kGatherThreads, 0, st>>>(a, tabs, few, a.n_rows);
        });
        SAR_LAUNCH_CHECK();
        a.n_rows = few;
        a.n_long = std::min(a.n_long, few);
        if (few == 0) return SAR_OK;
    }
    SAR_DISPATCH_LANES(T, a.F, a.ld, {
        auto fn = k_spmm_bwd_all<T, kG, kR>;
        static const int resident = resident_workgroups(fn);
        fn<<<persistent_grid_for(a.n_rows, a.n_long, resident), kGatherThreads, 0, st>>>(a, tabs);
    });
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

int check_row_shape(int dtype, int F)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    if (F <= 0) return sar::fail(SAR_ERR_INVALID_ARG, "F=%d must be positive", F);
    return SAR_OK;
}

// A wavefront covers 64 lane pieces of a row (1024 bytes; less where the row is so narrow that
// lanes have to move 8, 4 or 2 bytes); wider rows are processed as several launches over column
// ranges of about the same width, each seeing its slice of every row through the row stride.  No launch
// is narrower than a piece: its one lane would reach back into the columns of the launch before it.  What is
// left behind the last whole range (fp32 F = 16129: one value) takes a piece from that range instead.
struct ColumnChunks {
    int n, width;   // launches and values per launch (the last launch may be narrower)
    size_t fb;
    int piece;      // values per lane: 16 bytes' worth; rows that are narrower, the largest piece that divides them
    int lent;       // values the last launch takes over from the one before it: a piece or none
    int first(int c) const { return c * width - (c == n - 1 ? lent : 0); }
    int count(int c, int F) const { return (c == n - 1 ? F : first(c + 1)) - first(c); }
};

ColumnChunks column_chunks(int dtype, int F)
{
    ColumnChunks c;
    c.fb = dtype == SAR_F32 ? 4 : 2;
    const int full = dtype == SAR_F32 ? 4 : 8;
    c.piece = F >= full ? full : piece_for(dtype == SAR_F32, F);
    c.n = (F + 64 * c.piece - 1) / (64 * c.piece);
    c.width = ((F + c.n - 1) / c.n + c.piece - 1) / c.piece * c.piece;
    c.n = (F + c.width - 1) / c.width;
    c.lent = c.n > 1 && F - (c.n - 1) * c.width < c.piece ? c.piece : 0;
    return c;
}

template <typename P>
P* shift(P* p, size_t bytes)
{
    return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) + bytes) : nullptr;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

extern "C" int sar_spmm_block(const sar_blocks_t* b, int q, const void* Zq, int dtype, int F, float* acc,
                              void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_CHECK_ARG(q >= 0 && q < b->P, "block %d out of range [0,%d)", q, b->P);
    SAR_TRY(check_row_shape(dtype, F));
    const sar::Block& k = b->blk[q];
    if (k.n_rows == 0) return SAR_OK;
    SAR_CHECK_ARG(Zq && acc, "Zq or acc is null");
    SAR_CHECK_ARG(aligned16(Zq) && aligned16(acc), "Zq and acc must be 16-byte aligned");
    SpmmArgs a{};
    a.indptr = k.indptr;
    a.indices = reinterpret_cast<const uint32_t*>(k.indices);
    a.rows = reinterpret_cast<const uint32_t*>(k.rows);
    a.n_rows = k.n_rows;
    a.n_long = k.n_shared;
    a.ld = F;
    PtrTab tab{};
    const ColumnChunks cc = column_chunks(dtype, F);
    for (int c = 0; c < cc.n; ++c) {
        const size_t f0 = (size_t)cc.first(c);
        a.Z = shift(Zq, f0 * cc.fb);
        a.acc = acc + f0;
        a.F = cc.count(c, F);
        SAR_DISPATCH_ROW(dtype, cc.piece, SAR_TRY((launch_spmm<T, Mode::kBlock>(a, tab, 0, k.n_rows_wide, sar::as_stream(stream)))));
    }
    return SAR_OK;
}

namespace {

int check_act(int act)
{
    if (act != SAR_ACT_NONE && act != SAR_ACT_RELU)
        return sar::fail(SAR_ERR_UNSUPPORTED, "act %d is neither SAR_ACT_NONE nor SAR_ACT_RELU", act);
    return SAR_OK;
}

}  // namespace

extern "C" int sar_act_bwd(const void* h, const void* dH, int act, void* G, int dtype, int64_t count, void* stream)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    SAR_TRY(check_act(act));
    SAR_CHECK_ARG(count >= 0, "count=%lld is negative", (long long)count);
    if (count == 0) return SAR_OK;
    const int vec = piece_for(dtype == SAR_F32, (int)(count % 64 == 0 ? 64 : count % 64));
    SAR_CHECK_ARG(h && dH && G, "h, dH or G is null");
    SAR_CHECK_ARG(aligned16(h) && aligned16(dH) && aligned16(G), "h, dH and G must be 16-byte aligned");
    hipStream_t st = sar::as_stream(stream);
    if (act == SAR_ACT_NONE) {
        if (G != dH) SAR_HIP(hipMemcpyAsync(G, dH, (size_t)count * (dtype == SAR_F32 ? 4 : 2), hipMemcpyDeviceToDevice, st));
        return SAR_OK;
    }
    const int64_t n_vec = count / vec;
    const unsigned grid = (unsigned)std::min<int64_t>((n_vec + 255) / 256, 1 << 20);
    SAR_DISPATCH_ROW(dtype, vec, (k_act_bwd<T><<<grid, 256, 0, st>>>(static_cast<const T*>(h), static_cast<const T*>(dH),
                                                                     static_cast<T*>(G), n_vec)));
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

extern "C" int sar_spmm_end(const int32_t* deg, int mean, const float* acc, const void* residual, int act,
                            void* out, int dtype, int64_t n_dst, int F, void* stream)
{
    SAR_TRY(check_row_shape(dtype, F));
    SAR_TRY(check_act(act));
    SAR_CHECK_ARG(aligned16(residual), "residual must be 16-byte aligned");
    SAR_CHECK_ARG(n_dst >= 0, "n_dst is negative");
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(acc && out && (!mean || deg), "acc, out or deg is null");
    SAR_CHECK_ARG(aligned16(acc) && aligned16(out), "acc and out must be 16-byte aligned");
    const int vec = piece_for(dtype == SAR_F32, F);
    const unsigned grid = (unsigned)std::min<int64_t>((n_dst * (F / vec) + 255) / 256, 1 << 20);
    SAR_DISPATCH_ROW(dtype, vec, (k_spmm_end<T><<<grid, 256, 0, sar::as_stream(stream)>>>(
                                     deg, mean, acc, static_cast<const T*>(residual), act, static_cast<T*>(out), n_dst, F)));
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

extern "C" int sar_spmm_all(const sar_blocks_t* b, const void* const* Zq, int dtype, int F, int mean,
                            const void* residual, int act, void* out, void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_TRY(check_row_shape(dtype, F));
    SAR_TRY(check_act(act));
    SAR_CHECK_ARG(aligned16(residual), "residual must be 16-byte aligned");
    if (!b->f_indptr) return sar::fail(SAR_ERR_STATE, "handle was built without SAR_BUILD_FUSED");
    if (b->n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(Zq && out, "Zq or out is null");
    SAR_CHECK_ARG(aligned16(out), "out must be 16-byte aligned");
    for (int q = 0; q < b->P; ++q) {
        SAR_CHECK_ARG(Zq[q] != nullptr || b->blk[q].nnz == 0, "Zq[%d] is null", q);
        SAR_CHECK_ARG(aligned16(Zq[q]), "Zq[%d] must be 16-byte aligned", q);
    }
    hipStream_t st = sar::as_stream(stream);
    SpmmArgs a{};
    a.indptr = b->f_indptr;
    a.indices = b->f_indices;
    a.rows = reinterpret_cast<const uint32_t*>(b->f_rows);
    a.n_rows = b->n_dst;   // destinations without in-edges come last in the list and get 0
    a.n_long = b->n_f_shared;
    a.deg = b->deg;
    a.ld = F;
    a.tag_shift = b->tag_shift;
    a.mean = mean;
    const ColumnChunks cc = column_chunks(dtype, F);
    for (int c = 0; c < cc.n; ++c) {
        const size_t f0 = (size_t)cc.first(c);
        PtrTab tab{};
        for (int q = 0; q < b->P; ++q) tab.p[q] = shift(Zq[q], f0 * cc.fb);
        a.out = shift(out, f0 * cc.fb);
        a.res = residual ? shift(residual, f0 * cc.fb) : nullptr;
        a.act = act;
        a.F = cc.count(c, F);
        SAR_DISPATCH_ROW(dtype, cc.piece, SAR_TRY((launch_spmm<T, Mode::kAll>(a, tab, b->P, 0, st))));
    }
    return SAR_OK;
}

extern "C" int sar_spmm_bwd_block(const sar_blocks_t* b, int q, const void* G, int mean, int dtype, int F,
                                  void* dZq, void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_CHECK_ARG(q >= 0 && q < b->P, "block %d out of range [0,%d)", q, b->P);
    SAR_TRY(check_row_shape(dtype, F));
    const sar::Block& k = b->blk[q];
    if (!k.t_indptr) return sar::fail(SAR_ERR_STATE, "handle was built without SAR_BUILD_TRANSPOSE");
    if (k.n_src == 0 || (sar::skips_untouched(b->flags) && k.n_t_rows == 0)) return SAR_OK;
    SAR_CHECK_ARG((G || b->n_dst == 0) && dZq, "G or dZq is null");
    SAR_CHECK_ARG(aligned16(G) && aligned16(dZq), "G and dZq must be 16-byte aligned");
    hipStream_t st = sar::as_stream(stream);
    SpmmArgs a{};
    a.indptr = k.t_indptr;
    a.indices = reinterpret_cast<const uint32_t*>(k.t_indices);
    a.rows = reinterpret_cast<const uint32_t*>(k.t_rows);
    // sources without edges come last in the list and get 0, unless the handle skips them
    a.n_rows = sar::skips_untouched(b->flags) ? k.n_t_rows : k.n_src;
    a.out_rank = (b->flags & SAR_BUILD_COMPACT) ? k.t_rank : nullptr;
    a.n_long = k.n_t_shared;
    a.deg = b->deg;
    a.ld = F;
    a.mean = mean;
    PtrTab tab{};
    const ColumnChunks cc = column_chunks(dtype, F);
    for (int c = 0; c < cc.n; ++c) {
        const size_t f0 = (size_t)cc.first(c);
        a.Z = shift(G, f0 * cc.fb);
        a.out = shift(dZq, f0 * cc.fb);
        a.F = cc.count(c, F);
        SAR_DISPATCH_ROW(dtype, cc.piece, SAR_TRY((launch_spmm<T, Mode::kBackward>(a, tab, 0, k.n_t_wide, st))));
    }
    return SAR_OK;
}

extern "C" int sar_spmm_bwd_all(const sar_blocks_t* b, const void* G, int mean, int dtype, int F,
                                void* const* dZq, void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_TRY(check_row_shape(dtype, F));
    if (!b->ft_rows) return sar::fail(SAR_ERR_STATE, "handle was built without SAR_BUILD_TRANSPOSE");
    if (b->P > SAR_MAX_BLOCKS)
        return sar::fail(SAR_ERR_UNSUPPORTED, "an all-blocks call takes at most %d blocks, the handle has %d: use the "
                         "per-block calls", SAR_MAX_BLOCKS, b->P);
    int64_t n_src_total = 0;
    for (int q = 0; q < b->P; ++q) n_src_total += b->blk[q].n_src;
    if (n_src_total == 0) return SAR_OK;
    SAR_CHECK_ARG((G || b->n_dst == 0) && dZq, "G or dZq is null");
    SAR_CHECK_ARG(aligned16(G), "G must be 16-byte aligned");
    for (int q = 0; q < b->P; ++q) {
        if (b->blk[q].n_src == 0 || (sar::skips_untouched(b->flags) && b->blk[q].n_t_rows == 0)) continue;
        SAR_CHECK_ARG(dZq[q] && aligned16(dZq[q]), "dZq[%d] is null or not 16-byte aligned", q);
    }
    hipStream_t st = sar::as_stream(stream);
    SpmmArgs a{};
    a.rows = b->ft_rows;
    a.n_rows = sar::skips_untouched(b->flags) ? b->n_ft_rows : n_src_total;
    a.n_long = b->n_ft_shared;
    a.deg = b->deg;
    a.ld = F;
    a.mean = mean;
    a.tag_shift = b->tag_shift;
    const ColumnChunks cc = column_chunks(dtype, F);
    for (int c = 0; c < cc.n; ++c) {
        const size_t f0 = (size_t)cc.first(c);
        BwdAllTabs tabs{};
        for (int q = 0; q < b->P; ++q) {
            const sar::Block& k = b->blk[q];
            if (k.n_src == 0) continue;
            tabs.t_indptr[q] = k.t_indptr;
            tabs.t_indices[q] = reinterpret_cast<const uint32_t*>(k.t_indices);
            tabs.dZ[q] = shift(dZq[q], f0 * cc.fb);
            tabs.rank[q] = (b->flags & SAR_BUILD_COMPACT) ? k.t_rank : nullptr;
        }
        a.Z = shift(G, f0 * cc.fb);
        a.F = cc.count(c, F);
        SAR_DISPATCH_ROW(dtype, cc.piece, SAR_TRY(launch_spmm_bwd_all<T>(a, tabs, b->n_ft_wide, st)));
    }
    return SAR_OK;
}

extern "C" int sar_error_add(const void* Eq, const int32_t* t_rank, int accumulate, void* Ep, int dtype, int64_t n,
                             int F, void* stream)
{
    SAR_TRY(check_row_shape(dtype, F));
    SAR_CHECK_ARG(n >= 0, "n is negative");
    if (n == 0) return SAR_OK;
    SAR_CHECK_ARG(t_rank && Ep, "t_rank or Ep is null");
    SAR_CHECK_ARG(aligned16(Eq) && aligned16(Ep), "Eq and Ep must be 16-byte aligned");
    SAR_CHECK_ARG(Eq != Ep, "Eq and Ep must not alias");
    const int vec = piece_for(dtype == SAR_F32, F);
    const int64_t total = n * (F / vec);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, kMaxPersistentWGs * 4));
    hipStream_t st = sar::as_stream(stream);
    SAR_DISPATCH_ROW(dtype, vec, (k_error_add<T><<<grid, 256, 0, st>>>(static_cast<const T*>(Eq), t_rank, accumulate,
                                                                       static_cast<T*>(Ep), n, F)));
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}
