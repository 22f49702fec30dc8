// Fused, rematerialising attention kernels for GAT (Eq. 3; Sec. 3.3) with the
// running-maximum incremental softmax of Sec. 3.4, as row gathers on gfx950.
//
// Forward: one wavefront owns one destination row.  Per edge it reads the
// source's score half t_j and the source row z_j (16 bytes per lane, a 1 KiB
// row is one wave-wide load, several in flight), forms e = LeakyReLU(s_i+t_j)
// and folds exp(e - m) z_j into fp32 registers, rescaling when the running
// maximum m grows.  Nothing per edge is written to memory.
//
// Backward: the same gather, run over the source-major index: one wavefront
// owns one SOURCE row j, keeps z_j and t_j in registers, and for every
// destination i of j reads G_i and the per-destination record (s_i, L_i,
// delta_i), recomputes alpha = exp(e - L_i) and accumulates
// dZ_j += alpha G_i, dt_j += du in registers.  dZ_q is written once per row,
// coalesced, with no atomics; only the tiny ds[i,h] += du uses atomics.
//
// All exponentials are taken in base 2: scores are pre-multiplied by log2(e)
// (LeakyReLU commutes with a positive scale), so e2 = LeakyReLU(s2 + t2) and
// exp(e - m) = exp2(e2 - m2).
#include <algorithm>
#include <mutex>
#include <vector>

#include "gather_common.h"
#include "gat_f256.h"
#include "gat_slices.h"
#include "gat_joint.h"
#include "gat_slots.h"
#include "sar_internal.h"

namespace {

using namespace sar;

constexpr int kU = 4;   // edges in flight per lane group

struct PtrTab {
    const void* p[SAR_MAX_BLOCKS];
};

__device__ inline float leaky(float u, float slope) { return u > 0.f ? u : slope * u; }

// ------------------------------------------------------------------ forward

struct FwdArgs {
    const int32_t* indptr;
    const uint32_t* indices;
    const uint32_t* rows;
    int64_t n_rows, n_long;
    int64_t n_hub;       // call over all blocks: the first rows, where a large workgroup shares them (0: none does)
    int64_t n_wide;      // per-block call: rows of 8 edges and more, the head of the list
    const void* Z;       // per-block call: this block's source rows
    const float* t;      //                 and their score halves [n_src,H]; null: formed from a_l
    const float* a_l;    // [H,D], used only when the source score halves are not given
    const float* s;      // destination score halves [n_dst,H]
    float* m;            // running state (per-block calls), natural-log units
    float* l;
    float* acc;
    void* out;           // batched call: normalised output rows
    float* L;            //               and log-sum-exp [n_dst,H]
    int H, D, F;         // heads, head width and row width handled by this launch
    int ldz, ldh;        // strides between nodes of the feature rows / of the per-head arrays
    int tag_shift;
    float slope;
    int act;             // SAR_ACT_*: the non-linearity of Eq. 3 on the normalised rows (batched call)
};

template <int VEC>
struct SoftState {
    float m2;          // running maximum of e, in log2 units
    float l;           // running sum of exp(e - m)
    float acc[VEC];    // running sum of exp(e - m) z
};

template <int VEC>
__device__ inline void state_reset(SoftState<VEC>& st)
{
    st.m2 = -INFINITY;
    st.l = 0.f;
#pragma unroll
    for (int x = 0; x < VEC; ++x) st.acc[x] = 0.f;
}

// st <- st (+) other : the recursive aggregation property of Sec. 3.2 for the
// (max, denominator, numerator) triple.
template <int VEC>
__device__ inline void state_merge(SoftState<VEC>& st, float om2, float ol, const float (&oacc)[VEC])
{
    const float mn = fmaxf(st.m2, om2);
    const float ref = (mn == -INFINITY) ? 0.f : mn;
    const float ca = fast_exp2(st.m2 - ref), cb = fast_exp2(om2 - ref);
    st.l = st.l * ca + ol * cb;
#pragma unroll
    for (int x = 0; x < VEC; ++x) st.acc[x] = st.acc[x] * ca + oacc[x] * cb;
    st.m2 = mn;
}

// Folds the edges idx[beg,end) into st; this wavefront takes share `share`
// of `shares` of them.  s2 is the destination score half of this
// lane's head in log2 units.
template <typename T, int G, bool ALL>
__device__ inline void fwd_edges(SoftState<Vec<T>::N>& st, const FwdArgs& a, const GlobalPtr<const void>* ztab,
                                 const GlobalPtr<const float>* ttab, int beg, int end, int share, int shares,
                                 const LaneMap<T, G>& lm, float s2, const float (&al)[Vec<T>::N], bool fly,
                                 bool pow2)
{
    constexpr int VEC = Vec<T>::N;
    constexpr int SLOTS = kWave / G;
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    const int step = row_share(beg, end, share, shares);
    for (int cb = beg; cb < end; cb += step) {
        const int cnt = min(kWave, end - cb);
        const uint32_t mine = (lm.lane < cnt) ? a.indices[cb + lm.lane] : 0u;
        for (int k0 = 0; k0 < cnt; k0 += SLOTS * kU) {
            typename Vec<T>::Raw raw[kU];
            float e2[kU];
            bool ok[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const int ek = k0 + k * SLOTS + lm.slot;
                const uint32_t id = __shfl(mine, ek & (kWave - 1));
                raw[k] = Vec<T>::zero();
                e2[k] = 0.f;
                ok[k] = ek < cnt;
                if (ek < cnt) {
                    const uint32_t j = id & mask;
                    const T* zb;
                    const float* tb;
                    if constexpr (ALL) {
                        zb = ztab[id >> a.tag_shift].template as<const T>();
                        tb = ttab[id >> a.tag_shift];
                    } else {
                        zb = static_cast<const T*>(a.Z);
                        tb = a.t;
                    }
                    if (!fly) e2[k] = tb[(int64_t)j * a.ldh + lm.h];
                    if (lm.on) raw[k] = Vec<T>::load(zb + (int64_t)j * a.ldz + lm.gl * VEC);
                }
            }
            if (fly) {   // t_j = <a_l, z_j> from the row just gathered
#pragma unroll
                for (int k = 0; k < kU; ++k) {
                    float v[VEC];
                    Vec<T>::unpack(raw[k], v);
                    float c = 0.f;
#pragma unroll
                    for (int x = 0; x < VEC; ++x) c = fmaf(al[x], v[x], c);
                    e2[k] = pow2 ? group_sum_pow2(c, lm.lph) : group_sum_any(c, lm.head_first, lm.lph);
                }
            }
            float mx = st.m2;
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                // -inf marks an absent edge
                e2[k] = ok[k] ? leaky(fmaf(e2[k], kLog2e, s2), a.slope) : -INFINITY;
                mx = fmaxf(mx, e2[k]);
            }
            if (mx > st.m2) {
                const float c = fast_exp2(st.m2 - mx);   // st.m2 = -inf gives 0
                st.l *= c;
#pragma unroll
                for (int x = 0; x < VEC; ++x) st.acc[x] *= c;
                st.m2 = mx;
            }
            const float ref = (st.m2 == -INFINITY) ? 0.f : st.m2;
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const float p = fast_exp2(e2[k] - ref);
                float v[VEC];
                Vec<T>::unpack(raw[k], v);
                st.l += p;
#pragma unroll
                for (int x = 0; x < VEC; ++x) st.acc[x] = fmaf(p, v[x], st.acc[x]);
            }
        }
    }
}

template <typename T, int G>
__device__ inline void fwd_merge_slots(SoftState<Vec<T>::N>& st)
{
    constexpr int VEC = Vec<T>::N;
#pragma unroll
    for (int o = G; o < kWave; o <<= 1) {
        const float om2 = __shfl_xor(st.m2, o), ol = __shfl_xor(st.l, o);
        float oacc[VEC];
#pragma unroll
        for (int x = 0; x < VEC; ++x) oacc[x] = __shfl_xor(st.acc[x], o);
        state_merge<VEC>(st, om2, ol, oacc);
    }
}

template <typename T, int G, bool ALL, bool RELU>
__device__ inline void fwd_finish_row(SoftState<Vec<T>::N>& st, const FwdArgs& a, int i,
                                      const LaneMap<T, G>& lm)
{
    constexpr int VEC = Vec<T>::N;
    if (lm.slot != 0 || !lm.on) return;
    const int64_t o = (int64_t)i * a.ldz + lm.gl * VEC;
    if constexpr (ALL) {
        // the division by the normaliser (Sec. 3.2), and L = m + log l for the backward pass
        const float inv = st.l > 0.f ? 1.f / st.l : 0.f;
        float v[VEC];
        // the non-linearity is a template parameter: reading it from the arguments here, branch
        // or select, costs the gather loop above a fifth of its speed (measured on 2 x 100 rows)
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            v[x] = st.acc[x] * inv;
            if (RELU) v[x] = fmaxf(v[x], 0.f);
        }
        Vec<T>::store(static_cast<T*>(a.out) + o, v);
        if ((lm.gl % lm.lph) == 0)
            a.L[(int64_t)i * a.ldh + lm.h] = st.l > 0.f ? (st.m2 + fast_log2(st.l)) * kLn2 : -INFINITY;
    } else {
        store_f32<VEC>(a.acc + o, st.acc);
        if ((lm.gl % lm.lph) == 0) {
            a.m[(int64_t)i * a.ldh + lm.h] = st.m2 * kLn2;
            a.l[(int64_t)i * a.ldh + lm.h] = st.l;
        }
    }
}

template <typename T, int G, bool ALL, bool RELU>
__global__ __launch_bounds__(kGatherThreads) void k_gat_fwd(FwdArgs a, PtrTab ztab_arg, PtrTab ttab_arg,
                                                            int P)
{
    constexpr int VEC = Vec<T>::N;
    __shared__ GlobalPtr<const void> ztab[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<const float> ttab[SAR_MAX_BLOCKS];
    __shared__ float part_acc[kWavesPerWG][G][VEC];
    __shared__ float part_ml[kWavesPerWG][G][2];
    if constexpr (ALL) {
        if ((int)threadIdx.x < P) {
            ztab[threadIdx.x] = ztab_arg.p[threadIdx.x];
            ttab[threadIdx.x] = static_cast<const float*>(ttab_arg.p[threadIdx.x]);
        }
        __syncthreads();
    }
    const LaneMap<T, G> lm(a.F, a.H, a.D);
    const int wave = threadIdx.x / kWave;
    const bool fly = a.a_l != nullptr, pow2 = is_pow2(lm.lph);
    float al[VEC];
#pragma unroll
    for (int x = 0; x < VEC; ++x) al[x] = (fly && lm.on) ? a.a_l[lm.gl * VEC + x] : 0.f;

    auto load_state = [&](SoftState<VEC>& st, int i) {
        state_reset<VEC>(st);
        if constexpr (!ALL) {
            // the state carried from the previous blocks enters through lane group 0
            if (lm.slot == 0) {
                st.m2 = a.m[(int64_t)i * a.ldh + lm.h] * kLog2e;
                st.l = a.l[(int64_t)i * a.ldh + lm.h];
                if (lm.on) load_f32<VEC>(a.acc + (int64_t)i * a.ldz + lm.gl * VEC, st.acc);
            }
        }
    };

    for (int64_t r = blockIdx.x; r < a.n_long; r += gridDim.x) {
        const int i = (int)a.rows[r];
        const float s2 = a.s[(int64_t)i * a.ldh + lm.h] * kLog2e;
        SoftState<VEC> st;
        if (wave == 0)
            load_state(st, i);
        else
            state_reset<VEC>(st);
        fwd_edges<T, G, ALL>(st, a, ztab, ttab, a.indptr[i], a.indptr[i + 1], wave, kWavesPerWG, lm, s2, al, fly, pow2);
        fwd_merge_slots<T, G>(st);
        if (lm.slot == 0) {
#pragma unroll
            for (int x = 0; x < VEC; ++x) part_acc[wave][lm.gl][x] = st.acc[x];
            part_ml[wave][lm.gl][0] = st.m2;
            part_ml[wave][lm.gl][1] = st.l;
        }
        __syncthreads();
        if (wave == 0) {
            for (int w = 1; w < kWavesPerWG; ++w) {
                float oacc[VEC];
#pragma unroll
                for (int x = 0; x < VEC; ++x) oacc[x] = part_acc[w][lm.gl][x];
                state_merge<VEC>(st, part_ml[w][lm.gl][0], part_ml[w][lm.gl][1], oacc);
            }
            fwd_finish_row<T, G, ALL, RELU>(st, a, i, lm);
        }
        __syncthreads();
    }
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t r = a.n_long + from_behind(a.n_long, blockIdx.x, gridDim.x) * kWavesPerWG + wave; r < a.n_rows; r += n_waves) {
        const int i = (int)a.rows[r];
        const float s2 = a.s[(int64_t)i * a.ldh + lm.h] * kLog2e;
        SoftState<VEC> st;
        load_state(st, i);
        fwd_edges<T, G, ALL>(st, a, ztab, ttab, a.indptr[i], a.indptr[i + 1], 0, 1, lm, s2, al, fly, pow2);
        fwd_merge_slots<T, G>(st);
        fwd_finish_row<T, G, ALL, RELU>(st, a, i, lm);
    }
}

// ----------------------------------------------------------------- backward

struct BwdArgs {
    const int32_t* t_indptr[SAR_MAX_BLOCKS];   // per block (one entry for per-block calls)
    const int32_t* t_indices[SAR_MAX_BLOCKS];
    const void* Z[SAR_MAX_BLOCKS];
    const float* t[SAR_MAX_BLOCKS];
    void* dZ[SAR_MAX_BLOCKS];
    float* dt[SAR_MAX_BLOCKS];
    const int32_t* rank[SAR_MAX_BLOCKS];       // compact outputs: row of dZ / dt of source j (null: j)
};

struct BwdScalars {
    const uint32_t* rows;       // source work list; tagged with the block when ALL
    int64_t n_rows, n_long;
    int64_t n_wide;             // list entries [n_wide, n_rows) have few edges: several sources per wavefront
    int64_t n_touched;          // list entries [n_touched, n_rows) have no edge at all
    // all-blocks calls on a handle that lists them: the n_single list entries before n_touched are
    // the sources of ONE edge, also listed destination-major (destination, tagged source, error row)
    int64_t n_single;
    const int32_t* s_dst;
    const uint32_t* s_src;
    const int32_t* s_row;
    const int64_t* n_src_host;  // host: rows of every block's dZ_q / dt_q (null: unknown)
    int n_blocks;
    const void* G;              // [n_dst,H,D]
    const float4* rec;          // [n_dst,H]: (s*log2e, L*log2e, delta, unused)
    const float* a_l;           // [H,D]
    float* ds;                  // [n_dst,H], atomically accumulated: the array or the first of ds_copies copies
    int64_t ds_stride;          // values between copies
    int ds_copies;              // a power of two
    float* partial;             // [gridDim.x][F] per-workgroup da_l partial sums
    int H, D, F;
    int ldz, ldh;               // node strides of feature rows / per-head arrays
    int tag_shift;
    float slope;
    bool wide_done;             // the first n_wide list entries have been served (gat_slices.h)
};

template <int VEC>
struct BwdAcc {
    float dz[VEC];   // sum_i alpha G_i
    float dt;        // sum_i du   (this lane's head)
};

// Edges (destinations) idx[beg,end) of one source row.
template <typename T, int G>
__device__ inline void bwd_edges(BwdAcc<Vec<T>::N>& ac, const BwdScalars& a, const int32_t* idx, int beg,
                                 int end, int share, int shares, const LaneMap<T, G>& lm,
                                 const float (&zj)[Vec<T>::N], float t2, bool pow2)
{
    constexpr int VEC = Vec<T>::N;
    constexpr int SLOTS = kWave / G;
    const T* Gp = static_cast<const T*>(a.G);
    const int step = row_share(beg, end, share, shares);
    for (int cb = beg; cb < end; cb += step) {
        const int cnt = min(kWave, end - cb);
        const int mine = (lm.lane < cnt) ? idx[cb + lm.lane] : 0;
        for (int k0 = 0; k0 < cnt; k0 += SLOTS * kU) {
            typename Vec<T>::Raw raw[kU];
            float4 rec[kU];
            int dst[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const int ek = k0 + k * SLOTS + lm.slot;
                const int i = __shfl(mine, ek & (kWave - 1));
                dst[k] = (ek < cnt) ? i : -1;
                raw[k] = Vec<T>::zero();
                rec[k] = make_float4(0.f, INFINITY, 0.f, 0.f);   // L = +inf gives alpha = 0
                if (ek < cnt) {
                    rec[k] = a.rec[(int64_t)i * a.ldh + lm.h];
                    if (lm.on) raw[k] = Vec<T>::load(Gp + (int64_t)i * a.ldz + lm.gl * VEC);
                }
            }
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                float g[VEC];
                Vec<T>::unpack(raw[k], g);
                float c = 0.f;
#pragma unroll
                for (int x = 0; x < VEC; ++x) c = fmaf(g[x], zj[x], c);
                c = pow2 ? group_sum_pow2(c, lm.lph) : group_sum_any(c, lm.head_first, lm.lph);
                const float u2 = rec[k].x + t2;
                const float alpha = fast_exp2(leaky(u2, a.slope) - rec[k].y);
                const float de = alpha * (c - rec[k].z);
                const float du = u2 > 0.f ? de : a.slope * de;
#pragma unroll
                for (int x = 0; x < VEC; ++x) ac.dz[x] = fmaf(alpha, g[x], ac.dz[x]);
                ac.dt += du;
                if (dst[k] >= 0 && lm.on && (lm.gl % lm.lph) == 0)
                    unsafeAtomicAdd(a.ds + (int64_t)dst[k] * a.ldh + lm.h, du);
            }
        }
    }
}

template <typename T, int G>
__device__ inline void bwd_merge_slots(BwdAcc<Vec<T>::N>& ac)
{
#pragma unroll
    for (int o = G; o < kWave; o <<= 1) {
#pragma unroll
        for (int x = 0; x < Vec<T>::N; ++x) ac.dz[x] += __shfl_xor(ac.dz[x], o);
        ac.dt += __shfl_xor(ac.dt, o);
    }
}

template <typename T, int G, bool ALL>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd(BwdArgs tabs, BwdScalars a)
{
    constexpr int VEC = Vec<T>::N;
    __shared__ float part[kWavesPerWG][G][VEC + 1];
    const LaneMap<T, G> lm(a.F, a.H, a.D);
    const int wave = threadIdx.x / kWave;
    const bool pow2 = is_pow2(lm.lph);
    const uint32_t mask = ALL ? ((1u << a.tag_shift) - 1u) : 0xffffffffu;
    a.ds += (int64_t)(blockIdx.x & (unsigned)(a.ds_copies - 1)) * a.ds_stride;

    float al[VEC], dal[VEC];
#pragma unroll
    for (int x = 0; x < VEC; ++x) {
        al[x] = lm.on ? a.a_l[lm.gl * VEC + x] : 0.f;
        dal[x] = 0.f;
    }

    // Source row j of block q: z_j and t_j stay in registers for all its edges.
    auto row_inputs = [&](uint32_t id, int& q, int& j, float (&zj)[VEC], float& t2) {
        q = ALL ? (int)(id >> a.tag_shift) : 0;
        j = (int)(id & mask);
        typename Vec<T>::Raw r = Vec<T>::zero();
        if (lm.on) r = Vec<T>::load(static_cast<const T*>(tabs.Z[q]) + (int64_t)j * a.ldz + lm.gl * VEC);
        Vec<T>::unpack(r, zj);
        if (tabs.t[q]) {
            t2 = f256::score_log2(tabs.t[q][(int64_t)j * a.ldh + lm.h]);
        } else {
            float c = 0.f;
#pragma unroll
            for (int x = 0; x < VEC; ++x) c = fmaf(al[x], zj[x], c);
            t2 = f256::score_log2(pow2 ? group_sum_pow2(c, lm.lph) : group_sum_any(c, lm.head_first, lm.lph));
        }
    };
    // dZ_q[j] = sum alpha G + dt a_l ; dt_q[j] = dt ; da_l += dt z_j
    auto row_outputs = [&](const BwdAcc<VEC>& ac, int q, int j, const float (&zj)[VEC], int64_t jo) {
        if (lm.slot != 0 || !lm.on) return;
        float v[VEC];
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            v[x] = fmaf(ac.dt, al[x], ac.dz[x]);
            dal[x] = fmaf(ac.dt, zj[x], dal[x]);
        }
        Vec<T>::store(static_cast<T*>(tabs.dZ[q]) + jo * a.ldz + lm.gl * VEC, v);
        if ((lm.gl % lm.lph) == 0 && tabs.dt[q]) tabs.dt[q][jo * a.ldh + lm.h] = ac.dt;
    };

    for (int64_t r = blockIdx.x; r < a.n_long; r += gridDim.x) {
        int q, j;
        float zj[VEC], t2;
        row_inputs(a.rows[r], q, j, zj, t2);
        BwdAcc<VEC> ac = {};
        bwd_edges<T, G>(ac, a, tabs.t_indices[q], tabs.t_indptr[q][j], tabs.t_indptr[q][j + 1], wave,
                        kWavesPerWG, lm, zj, t2, pow2);
        bwd_merge_slots<T, G>(ac);
        if (lm.slot == 0) {
#pragma unroll
            for (int x = 0; x < VEC; ++x) part[wave][lm.gl][x] = ac.dz[x];
            part[wave][lm.gl][VEC] = ac.dt;
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int x = 0; x <= VEC; ++x) {
                float s = 0.f;
                for (int w = 0; w < kWavesPerWG; ++w) s += part[w][lm.gl][x];
                if (x < VEC)
                    ac.dz[x] = s;
                else
                    ac.dt = s;
            }
            row_outputs(ac, q, j, zj, tabs.rank[q] ? (int64_t)tabs.rank[q][j] : (int64_t)j);
        }
        __syncthreads();
    }
    // One source per wavefront.  Most sources of a partitioned graph have a handful of edges, so
    // what a wavefront spends its time on is the chain list entry -> edge range -> indices -> rows;
    // the first two links (and the output row) of the NEXT source are read while this one is
    // processed, the list entry of the one after that as well.
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    int64_t r = a.n_long + from_behind(a.n_long, blockIdx.x, gridDim.x) * kWavesPerWG + wave;
    struct Ahead {
        uint32_t id;
        int beg, end;
        int64_t jo;
    };
    auto look_up = [&](uint32_t id) {
        Ahead m;
        m.id = id;
        const int q = ALL ? (int)(id >> a.tag_shift) : 0, j = (int)(id & mask);
        m.beg = tabs.t_indptr[q][j];
        m.end = tabs.t_indptr[q][j + 1];
        m.jo = tabs.rank[q] ? (int64_t)tabs.rank[q][j] : (int64_t)j;
        return m;
    };
    Ahead next{};
    uint32_t id_after = 0;
    if (r < a.n_rows) next = look_up(a.rows[r]);
    if (r + n_waves < a.n_rows) id_after = a.rows[r + n_waves];
    for (; r < a.n_rows; r += n_waves) {
        const Ahead cur = next;
        if (r + n_waves < a.n_rows) next = look_up(id_after);
        if (r + 2 * n_waves < a.n_rows) id_after = a.rows[r + 2 * n_waves];
        int q, j;
        float zj[VEC], t2;
        row_inputs(cur.id, q, j, zj, t2);
        BwdAcc<VEC> ac = {};
        bwd_edges<T, G>(ac, a, tabs.t_indices[q], cur.beg, cur.end, 0, 1, lm, zj, t2, pow2);
        bwd_merge_slots<T, G>(ac);
        row_outputs(ac, q, j, zj, cur.jo);
    }

    // this workgroup's share of da_l = sum_j dt_j z_j
    __syncthreads();
    if (lm.slot == 0)
#pragma unroll
        for (int x = 0; x < VEC; ++x) part[wave][lm.gl][x] = dal[x];
    __syncthreads();
    if (wave == 0 && lm.slot == 0 && lm.on) {
        float v[VEC];
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            float s = 0.f;
            for (int w = 0; w < kWavesPerWG; ++w) s += part[w][lm.gl][x];
            v[x] = s;
        }
        store_f32<VEC>(a.partial + (int64_t)blockIdx.x * a.F + lm.gl * VEC, v);
    }
}

// out(x) += sum_w partial[w ld + x] for the COLS values x of a workgroup: eight rows' loads a thread under way at a time,
// then the wavefronts' sums, one barrier.
template <int COLS, typename Out>
__device__ inline void add_columns(const float* __restrict__ partial, int n_part, int64_t ld, Out out)
{
    __shared__ float red[kWavesPerWG][COLS];
    float sum[COLS] = {};
    float* const to = threadIdx.x < COLS ? out((int)threadIdx.x) : nullptr;
    const float was = to ? *to : 0.f;
    constexpr int kRows = 8;
    for (int w0 = threadIdx.x; w0 < n_part; w0 += 256 * kRows) {
        float v[kRows][COLS];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int w = w0 + 256 * r;
#pragma unroll
            for (int x = 0; x < COLS; ++x) v[r][x] = 0.f;
            if (w >= n_part) continue;
            if constexpr (COLS == 4)
                load_f32<4>(partial + w * ld, v[r]);
            else
                v[r][0] = partial[w * ld];
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int x = 0; x < COLS; ++x) sum[x] += v[r][x];
    }
#pragma unroll
    for (int x = 0; x < COLS; ++x) {
        const float s = f256::group_all<kWave, f256::OpSum>(sum[x]);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave][x] = s;
    }
    __syncthreads();
    if (!to) return;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerWG; ++w) s += red[w][threadIdx.x];
    *to = was + s;
}

// Columns a workgroup sums: a cache line of four wanted bytes a row is nothing while the rows are few (243 of them, 128
// columns 3.8 us, by fours 2.6), and beyond that the chip wants the workgroups (2048 rows, 256 columns: 8.5 us by fours 9).
constexpr int kFewPartials = 512;

// out[f] += sum_w partial[w][f]
template <int COLS>
__global__ __launch_bounds__(256) void k_reduce_partials(const float* __restrict__ partial, int n_part, int F,
                                                         float* __restrict__ out)
{
    const int f0 = blockIdx.x * COLS;
    add_columns<COLS>(partial + f0, n_part, F, [&](int x) { return out + f0 + x; });
}
int reduce_partials(const float* partial, int n_part, int F, float* out, hipStream_t st)
{
    if (F % 4 == 0 && n_part <= kFewPartials)      // (rows of whole 16 bytes: the scratch is aligned)
        k_reduce_partials<4><<<F / 4, 256, 0, st>>>(partial, n_part, F, out);
    else
        k_reduce_partials<1><<<F, 256, 0, st>>>(partial, n_part, F, out);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// ---------------------------------------------------------------- node-wise

// Lanes of the node-wise kernels: a head is LPH lanes of VEC values (the power of two that covers
// it; lanes behind its end idle), a node is the launch's H heads, a wavefront takes as many nodes
// (slots) as fit.  RAG: head widths that are no multiple of 4, with the last lane of a head on the
// head's last four values as in gat_slots.h (`dup` of them are the lane before it's), and heads of
// fewer than 4 values moved one by one.
template <typename T, int VEC, int LPH, bool RAG>
struct NodeLanes {
    int lane, k_pos, slot, n_slots, h, foff, dup, width;
    bool on;
    __device__ inline NodeLanes(int H, int D)
    {
        lane = threadIdx.x & (kWave - 1);
        k_pos = lane % LPH;
        const int grp = lane / LPH;
        n_slots = (kWave / LPH) / H;
        slot = grp / H;
        h = grp - slot * H;
        width = D;
        on = slot < n_slots && VEC * k_pos < D;
        const int off = RAG ? max(0, min(VEC * k_pos, D - VEC)) : VEC * k_pos;
        dup = (RAG && on) ? VEC * k_pos - off : 0;
        foff = h * D + off;
    }
    __device__ inline void load(const T* row, float (&v)[VEC]) const
    {
        if constexpr (!RAG) {
            if constexpr (VEC == Vec<T>::N)
                Vec<T>::unpack(Vec<T>::load(row + foff), v);
            else
                f256::Row4<T>::unpack(f256::load_raw<T, false>(row + foff), v);
        } else {
            if (width >= VEC) {
                f256::Row4<T>::unpack(f256::load_raw<T, true>(row + foff), v);
            } else {
#pragma unroll
                for (int x = 0; x < VEC; ++x) v[x] = x < width ? widen(row[foff + x]) : 0.f;
            }
        }
    }
    __device__ inline void store(T* row, const float (&v)[VEC]) const
    {
        if constexpr (!RAG) {
            if constexpr (VEC == Vec<T>::N)
                Vec<T>::store(row + foff, v);
            else
                f256::store4<T, false>(row + foff, v);
        } else {
            if (width >= VEC) {
                f256::store4<T, true>(row + foff, v);
            } else {
#pragma unroll
                for (int x = 0; x < VEC; ++x)
                    if (x < width) narrow(row + foff + x, v[x]);
            }
        }
    }
    __device__ inline void load_vec(const float* p, float (&v)[VEC]) const     // fp32 rows
    {
#pragma unroll
        for (int x = 0; x < VEC; ++x) v[x] = x < width ? p[foff + x] : 0.f;
    }
    // whether this lane (and not the one before it) speaks for its value x
    __device__ inline bool owns(int x) const { return !RAG || (x >= dup && x < width); }
    __device__ inline float head_sum(float v) const { return f256::group_all<LPH, f256::OpSum>(v); }
    // The sum from the head's first lane to its last, one after the other; the last lane has it.
    __device__ inline float head_sum_in_order(float v) const
    {
        float s = v;
        for (int k = VEC; k < width; k += VEC)
            s = __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x138 /* lane - 1 */, 0xf, 0xf, false)) + v;
        return s;
    }
    static __device__ inline float widen(float x) { return x; }
    static __device__ inline float widen(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }
    static __device__ inline void narrow(float* p, float v) { *p = v; }
    static __device__ inline void narrow(bf16_t* p, float v) { p->bits = (uint16_t)f32_to_bf16_rne(v); }
};

// a0 z0 + a1 z1 + a2 z2 with every product rounded before it is added.
__device__ inline float sum_of_three(const float* a, const float* z)
{
#pragma clang fp contract(off)
    const float p0 = a[0] * z[0], p1 = a[1] * z[1], p2 = a[2] * z[2];
    return p0 + p1 + p2;
}

// score[v,h] = <a[h], Z[v,h]>; one lane group per (node, head).  A second vector / output pair may
// ride along (the two halves of the attention score from one pass over Z); avec2 = null: only the first.
template <typename T, int VEC, int LPH, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_scores(const T* __restrict__ Z, int64_t n, int H, int D,
                                                           int ldz, int ldh,
                                                           const float* __restrict__ avec,
                                                           float* __restrict__ score,
                                                           const float* __restrict__ avec2,
                                                           float* __restrict__ score2)
{
    const NodeLanes<T, VEC, LPH, RAG> lm(H, D);
    // Heads of whole lanes that fill no power of two add lane after lane, the others pairwise.  (A score's last
    // bit decides on which side of LeakyReLU's kink an edge within rounding of zero falls: a shape's order of
    // addition is not to change.)
    const bool in_order = !RAG && !is_pow2(D / VEC);
    const int writer = in_order ? D / VEC - 1 : 0;
    float av[VEC] = {}, av2[VEC] = {};
    if (lm.on) {
        lm.load_vec(avec, av);
        if (avec2) lm.load_vec(avec2, av2);
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            av[x] = lm.owns(x) ? av[x] : 0.f;
            av2[x] = lm.owns(x) ? av2[x] : 0.f;
        }
    }
    const int64_t wave_id = ((int64_t)blockIdx.x * kGatherThreads + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t v0 = wave_id * lm.n_slots; v0 < n; v0 += n_waves * lm.n_slots) {
        const int64_t v = v0 + lm.slot;
        float z[VEC] = {};
        if (v < n && lm.on) lm.load(Z + v * ldz, z);
        float c = 0.f, c2 = 0.f;
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            z[x] = lm.owns(x) ? z[x] : 0.f;      // not only a: an infinity the lane before owns is not 0 x inf here
            c = fmaf(av[x], z[x], c);
            c2 = fmaf(av2[x], z[x], c2);
        }
        if constexpr (RAG && LPH == 1) {
            if (D == 3) {                        // the aggregation kernels move such heads value by value
                c = sum_of_three(av, z);
                c2 = sum_of_three(av2, z);
            }
        }
        c = in_order ? lm.head_sum_in_order(c) : lm.head_sum(c);
        if (avec2) c2 = in_order ? lm.head_sum_in_order(c2) : lm.head_sum(c2);
        if (v < n && lm.on && lm.k_pos == writer) {
            score[v * ldh + lm.h] = c;
            if (avec2) score2[v * ldh + lm.h] = c2;
        }
    }
}

// The same for heads that no wavefront covers: one thread per (node, head), element-wise reads.
// Scores only; the aggregation kernels do not take such rows.
template <typename T>
__global__ __launch_bounds__(256) void k_scores_any(const T* __restrict__ Z, int64_t n, int H, int D,
                                                    const float* __restrict__ avec, float* __restrict__ score,
                                                    const float* __restrict__ avec2, float* __restrict__ score2)
{
    const int64_t total = n * H;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < total; k += (int64_t)gridDim.x * 256) {
        const int h = (int)(k % H);
        const T* z = Z + k * D;
        float c = 0.f, c2 = 0.f;
        for (int d = 0; d < D; ++d) {
            const float v = NodeLanes<T, 4, 4, true>::widen(z[d]);
            c = fmaf(avec[h * D + d], v, c);
            if (avec2) c2 = fmaf(avec2[h * D + d], v, c2);
        }
        score[k] = c;
        if (avec2) score2[k] = c2;
    }
}

__global__ __launch_bounds__(256) void k_fwd_begin(float* __restrict__ m, float* __restrict__ l,
                                                   float* __restrict__ acc, int64_t n_h, int64_t n_f)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n_f; k += (int64_t)gridDim.x * 256) {
        acc[k] = 0.f;
        if (k < n_h) {
            m[k] = -INFINITY;
            l[k] = 0.f;
        }
    }
}

template <typename T, int VEC, int LPH, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_fwd_end(const float* __restrict__ m,
                                                            const float* __restrict__ l,
                                                            const float* __restrict__ acc, T* __restrict__ out,
                                                            float* __restrict__ L, int64_t n, int H, int D,
                                                            int ldz, int ldh, int act)
{
    const NodeLanes<T, VEC, LPH, RAG> lm(H, D);
    const int64_t wave_id = ((int64_t)blockIdx.x * kGatherThreads + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t v0 = wave_id * lm.n_slots; v0 < n; v0 += n_waves * lm.n_slots) {
        const int64_t v = v0 + lm.slot;
        if (v >= n || !lm.on) continue;
        const float lv = l[v * ldh + lm.h];
        const float inv = lv > 0.f ? 1.f / lv : 0.f;
        float a[VEC];
        if constexpr (RAG)
            lm.load_vec(acc + v * ldz, a);
        else
            load_f32<VEC>(acc + v * ldz + lm.foff, a);
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            a[x] *= inv;
            if (act == SAR_ACT_RELU) a[x] = fmaxf(a[x], 0.f);
        }
        lm.store(out + v * ldz, a);
        if (lm.k_pos == 0)
            L[v * ldh + lm.h] = lv > 0.f ? m[v * ldh + lm.h] + fast_log2(lv) * kLn2 : -INFINITY;
    }
}

// rec[i,h] = (s log2e, L log2e, <G_i, out_i>, 0) and ds = 0.  With a non-linearity, `out` holds
// h = act(aggregate) and Gr the error of h: the error of the aggregate, Gr * act'(.), is formed
// here from h alone (ReLU: h > 0 exactly where the aggregate is, and there they are equal, so
// <G_i, out_i> is unchanged) and written to Gact for the block kernels to gather.  (Gact may be Gr
// itself: lanes that share values of a ragged head read them before either writes, in one
// instruction each, and write the same bits.)
template <typename T, int VEC, int LPH, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_bwd_begin(const T* Gr, const T* __restrict__ out,
                                                              const float* __restrict__ s,
                                                              const float* __restrict__ L, float4* __restrict__ rec,
                                                              float* __restrict__ ds, int64_t n, int H, int D,
                                                              int ldz, int ldh, int act, T* Gact)
{
    const NodeLanes<T, VEC, LPH, RAG> lm(H, D);
    const int64_t wave_id = ((int64_t)blockIdx.x * kGatherThreads + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t v0 = wave_id * lm.n_slots; v0 < n; v0 += n_waves * lm.n_slots) {
        const int64_t v = v0 + lm.slot;
        float g[VEC] = {}, o[VEC] = {};
        if (v < n && lm.on) {
            lm.load(Gr + v * ldz, g);
            lm.load(out + v * ldz, o);
            if (act == SAR_ACT_RELU) {
#pragma unroll
                for (int x = 0; x < VEC; ++x) g[x] = o[x] > 0.f ? g[x] : 0.f;
                lm.store(Gact + v * ldz, g);
            }
        }
        float c = 0.f;
#pragma unroll
        for (int x = 0; x < VEC; ++x) c = lm.owns(x) ? fmaf(g[x], o[x], c) : c;
        c = lm.head_sum(c);
        if (v < n && lm.on && lm.k_pos == 0) {
            const int64_t k = v * ldh + lm.h;
            rec[k] = make_float4(s[k] * kLog2e, L[k] * kLog2e, c, 0.f);
            ds[k] = 0.f;
        }
    }
}

// dZdst[i] = ds[i] a_r (+ dZadd[i]) ; per-workgroup partial of da_r = sum_i ds[i] Zdst[i]
template <typename T, int VEC, int LPH, bool RAG>
__global__ __launch_bounds__(kGatherThreads) void k_bwd_end(const T* __restrict__ Zdst, const float* __restrict__ ds,
                                                            const float* __restrict__ a_r, const T* dZadd,
                                                            const int32_t* __restrict__ add_rank, T* dZdst,
                                                            float* __restrict__ partial, int64_t n, int H, int D,
                                                            int ldz, int ldh)
{
    __shared__ float part[kWavesPerWG][kWave][VEC];
    const NodeLanes<T, VEC, LPH, RAG> lm(H, D);
    const int wave = threadIdx.x / kWave;
    float ar[VEC] = {}, dar[VEC] = {};
    if (lm.on) lm.load_vec(a_r, ar);
    const int64_t wave_id = (int64_t)blockIdx.x * kWavesPerWG + wave;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerWG;
    for (int64_t v0 = wave_id * lm.n_slots; v0 < n; v0 += n_waves * lm.n_slots) {
        const int64_t v = v0 + lm.slot;
        if (v >= n || !lm.on) continue;
        const float d = ds[v * ldh + lm.h];
        float z[VEC], o[VEC] = {};
        lm.load(Zdst + v * ldz, z);
        int64_t va = v;
        bool add = dZadd != nullptr && dZdst != nullptr;
        if (add && add_rank) {
            va = add_rank[v];
            add = add_rank[v + 1] > (int32_t)va;
        }
        if (add) lm.load(dZadd + va * ldz, o);
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
            o[x] = fmaf(d, ar[x], o[x]);
            dar[x] = fmaf(d, z[x], dar[x]);
        }
        if (dZdst) lm.store(dZdst + v * ldz, o);     // null: only da_r is wanted
    }
#pragma unroll
    for (int x = 0; x < VEC; ++x) part[wave][lm.lane][x] = dar[x];
    __syncthreads();
    // a thread per value of a node's lanes: a wavefront that summed its slots' values one after the other waited for LDS 128
    // times (4 heads of 32 bf16 values on a thousand nodes: the kernel 9.8 us, now 3.9)
    const int lanes = H * LPH;
    for (int t = threadIdx.x; t < lanes * VEC; t += kGatherThreads) {
        const int l = t / VEC, x = t % VEC, first = VEC * (l % LPH);
        const int off = RAG ? max(0, min(first, D - VEC)) : first;      // as in NodeLanes
        if (first >= D || off + x < first || off + x >= D) continue;
        float s = 0.f;
        for (int w = 0; w < kWavesPerWG; ++w) {
#pragma unroll 4
            for (int sl = 0; sl < lm.n_slots; ++sl) s += part[w][sl * lanes + l][x];
        }
        partial[(int64_t)blockIdx.x * (H * D) + l / LPH * D + off + x] = s;
    }
}

// --------------------------------------------------------------- host side

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_act(int act)
{
    if (act != SAR_ACT_NONE && act != SAR_ACT_RELU)
        return sar::fail(SAR_ERR_UNSUPPORTED, "act %d is neither SAR_ACT_NONE nor SAR_ACT_RELU", act);
    return SAR_OK;
}

int check_shape(int dtype, int H, int D)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    if (H <= 0 || D <= 0) return sar::fail(SAR_ERR_INVALID_ARG, "H and D must be positive (H=%d, D=%d)", H, D);
    // a head is covered by lanes that each move the largest piece (16, 8, 4 or 2 bytes) dividing it
    const int piece = piece_for(dtype == SAR_F32, D);
    if (D / piece > 64)
        return sar::fail(SAR_ERR_UNSUPPORTED, "one head of D=%d values in pieces of %d needs more than the 64 lanes "
                         "of a wavefront", D, piece);
    return SAR_OK;
}

int pow2_at_least(int x)
{
    int p = 1;
    while (p < x) p *= 2;
    return p;
}

// Which gather kernels take a launch.  All but the generic ones give a head LPH lanes of 4 values,
// the power of two >= D/4, which makes 64/LPH lane groups in a wavefront.
//   exact   rows of 256 contiguous values, every lane busy (gat_f256.h);
//   padded  the launch's heads need more than half of the lane groups (gat_f256.h; D a multiple of 4,
//           LPH 8..64): lanes behind a head's end and groups without a head idle.  The gathers are
//           bound by memory, not by lanes, so they cost little;
//   slots   they need half of the groups or fewer, or the head width is no multiple of 4, or a head
//           is four lanes (gat_slots.h): the groups left over take other edges.
//   generic heads of 1 to 3 values and bf16 heads of more than 256; in the forward pass also layers of two
//           kinds.  (Times in us, generic kernel/the others, of one call over all blocks on a share of 7.3M edges,
//           24 a row, and on one of 7.4M, 6 a row; "shipped": with the sources' score halves given.)
//           - heads of 4 or 8 values, which two lanes of 16 bytes hold where a slots head has four.  With score halves
//             formed in flight up to 4 such heads are better off in the slots' longer batches: fp32 4 x 4
//             241/232, 813/579, 4 x 8 283/257, 870/598, bf16 1 x 8 274/166, 913/551 (block by block 1 x 8 fp32
//             1056/719, 4 x 4 989/706); more heads are not: fp32 16 x 4 390/730, 970/1228, 8 x 8 401/445,
//             1001/855, bf16 16 x 8 421/733, 1061/1230.  Shipped, the generic kernel reads one value per head and
//             edge with no sum to form: on 75 thousand rows of 29, fp32 4 x 8 96/136, bf16 4 x 4 74/133, 1 x 4 66/64.
//           - bf16 layers of up to 512 values whose heads would fall into launches of different sizes, which one
//             generic launch takes whole: shipped 5 x 64 988/1506, 7 x 48 1090/1667, 3 x 96 966/1522; block by block
//             5 x 64 2272/2887; in flight 5 x 40 855/1038, 1525/2052, 9 x 24 755/1148, 1451/2236, 25 x 16 1273/1699,
//             1985/2907, 7 x 72 2168/2572, 3178/4994.  In flight over all blocks two launches win where the
//             generic kernel's row needs a whole wavefront and its heads a sum lane after lane (no power of
//             two of lanes): 7 x 48 1704/1248, 2526/2388, 5 x 56 1797/1205, 2621/2325, 3 x 96 2416/1272, 3442/2378,
//             3 x 120 2887/1418, 4003/2650; not 5 x 64 (1422/1148, 2147/2195) and 3 x 80 (1149/1219, 1849/2363).
// (Where two slots fit, the padded kernel reads as fast on large graphs, 4 x 32 fp32 on 7.4M edges 603 us and 608, but a long
// row takes it twice as many round trips: 1 x 128 bf16, 2.2M edges, given scores 237 us and 176 with slots, 4 x 32 bf16 on 2000
// rows of 88 33.9 and 26.0, block by block on 136 thousand edges 29 and 25.)
enum class Gather { kGeneric, kExact, kPadded, kSlots };
struct LaunchGeo {
    Gather kind;
    int lph, n_slots;
    bool ragged;
};

// Heads of width D a wavefront of the slots kernels (and of the padded ones) has lane groups for.
int lane_groups(int D) { return 64 / std::max(4, pow2_at_least((D + 3) / 4)); }

// What a launch is for: the forward pass with the sources' score halves given, or formed in flight for
// one block or for all; or the backward pass.
enum class Pass { kFwdShipped, kFwdBlock, kFwdAll, kBwd };
Pass fwd_pass(bool shipped, bool all) { return shipped ? Pass::kFwdShipped : all ? Pass::kFwdAll : Pass::kFwdBlock; }

bool generic_layer(int dtype, int H, int D, Pass pass)
{
    if (D < 4 || D > 256) return true;
    if (pass == Pass::kBwd) return false;
    if (D == 4 || D == 8) return H > 4 || pass == Pass::kFwdShipped;
    const int n = (H + lane_groups(D) - 1) / lane_groups(D);
    if (dtype != SAR_BF16 || D % 8 != 0 || H % n == 0 || H * D > 512) return false;
    return pass != Pass::kFwdAll || n > 2 || H * D <= 256 || D <= 32 || is_pow2(D / 8);
}

LaunchGeo launch_geo(int dtype, int Hg, int D, int ldz, Pass pass)
{
    if (generic_layer(dtype, ldz / D, D, pass)) return LaunchGeo{Gather::kGeneric, 0, 0, false};
    const int lph = std::max(4, pow2_at_least((D + 3) / 4)), groups = 64 / lph;
    if (Hg * lph == 64 && D == 4 * lph && ldz == f256::kF) return LaunchGeo{Gather::kExact, lph, 1, false};
    int slots = 1;
    while (slots * 2 * Hg <= groups) slots *= 2;
    if (D % 4 == 0) {
        if (slots == 1 && lph >= 8) return LaunchGeo{Gather::kPadded, lph, 1, false};
    }
    return LaunchGeo{Gather::kSlots, lph, slots, D % 4 != 0};
}

// Heads are independent in Eq. 3, so a layer of more heads than a wavefront has lane groups for is
// processed as several launches over groups of heads, as even as they come, each launch seeing its
// slice of every row through the row stride.
struct HeadGroups {
    int n, most, H;      // launches, heads of a launch at most, heads of the layer
    size_t fb;           // bytes per feature value
    int first(int g) const { return g * most; }
    int count(int g) const { return std::min(most, H - g * most); }
};

HeadGroups head_groups(int dtype, int H, int D, Pass pass)
{
    HeadGroups g;
    g.H = H;
    g.fb = dtype == SAR_F32 ? 4 : 2;
    const int groups = generic_layer(dtype, H, D, pass) ? std::max(1, 64 * piece_for(dtype == SAR_F32, D) / D)
                                                           : lane_groups(D);
    g.n = (H + groups - 1) / groups;
    g.most = (H + g.n - 1) / g.n;
    g.n = (H + g.most - 1) / g.most;
    return g;
}

// Geometry of the node-wise kernels (NodeLanes): 16 bytes per lane where the head width is whole
// 16-byte pieces, else 4 values.
struct NodeGeo {
    int vec, lph;
    bool ragged;
    HeadGroups hg;
    int slots(int g) const { return (kWave / lph) / hg.count(g); }
};

NodeGeo node_geo(int dtype, int H, int D)
{
    NodeGeo g;
    const int full = dtype == SAR_F32 ? 4 : 8;
    g.vec = D % full == 0 ? full : 4;
    g.ragged = D % 4 != 0;
    g.lph = pow2_at_least((D + g.vec - 1) / g.vec);
    g.hg.H = H;
    g.hg.fb = dtype == SAR_F32 ? 4 : 2;
    const int groups = 64 / g.lph;
    g.hg.n = (H + groups - 1) / groups;
    g.hg.most = (H + g.hg.n - 1) / g.hg.n;
    g.hg.n = (H + g.hg.most - 1) / g.hg.most;
    return g;
}

#define SAR_NODE_LPH(geo, ...)                                          \
    switch ((geo).lph) {                                                \
        case 1: { constexpr int kL = 1; __VA_ARGS__; } break;           \
        case 2: { constexpr int kL = 2; __VA_ARGS__; } break;           \
        case 4: { constexpr int kL = 4; __VA_ARGS__; } break;           \
        case 8: { constexpr int kL = 8; __VA_ARGS__; } break;           \
        case 16: { constexpr int kL = 16; __VA_ARGS__; } break;         \
        case 32: { constexpr int kL = 32; __VA_ARGS__; } break;         \
        default: { constexpr int kL = 64; __VA_ARGS__; } break;         \
    }
// Runs `...` with T, kV, kL, kR bound to the row type, VEC, LPH and RAG of `geo`.
#define SAR_DISPATCH_NODE(dtype, geo, ...)                              \
    do {                                                                \
        if ((dtype) == SAR_F32) {                                       \
            using T = float;                                            \
            constexpr int kV = 4;                                       \
            if ((geo).ragged) {                                         \
                constexpr bool kR = true;                               \
                SAR_NODE_LPH(geo, __VA_ARGS__);                         \
            } else {                                                    \
                constexpr bool kR = false;                              \
                SAR_NODE_LPH(geo, __VA_ARGS__);                         \
            }                                                           \
        } else {                                                        \
            using T = bf16_t;                                           \
            if ((geo).vec == 8) {                                       \
                constexpr int kV = 8;                                   \
                constexpr bool kR = false;                              \
                SAR_NODE_LPH(geo, __VA_ARGS__);                         \
            } else if ((geo).ragged) {                                  \
                constexpr int kV = 4;                                   \
                constexpr bool kR = true;                               \
                SAR_NODE_LPH(geo, __VA_ARGS__);                         \
            } else {                                                    \
                constexpr int kV = 4;                                   \
                constexpr bool kR = false;                              \
                SAR_NODE_LPH(geo, __VA_ARGS__);                         \
            }                                                           \
        }                                                               \
    } while (0)

template <typename P>
P* shift(P* p, size_t bytes)
{
    return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) + bytes) : nullptr;
}

unsigned persistent_grid(int64_t n_rows, int64_t n_long)
{
    const int64_t want = n_long + (n_rows - n_long + kWavesPerWG - 1) / kWavesPerWG;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, kMaxPersistentWGs));
}

unsigned nodewise_grid(int64_t n, int slots, int64_t most = kMaxPersistentWGs)
{
    const int64_t waves = (n + slots - 1) / slots;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((waves + kWavesPerWG - 1) / kWavesPerWG, most));
}

// k_bwd_begin reads two arrays and keeps nothing from row to row, so a wavefront may as well take its rows once, by workgroups that
// come in the rows' order: walked by a resident grid the rows under way lie far apart, which memory answers more slowly.  Against it
// stands what starting workgroups costs.  That decides for a launch that moves little more than fits the 256 MiB memory-side cache, for
// wavefronts that move little at a time, and for rows of unaligned pieces.
// Bytes are counted with the records, s, L and ds.  us, resident / once, where the call before has read the arrays and where they are in
// no cache: fp32 4 x 64, 169 MiB 30 / 32, 65 / 63; 295 MiB 54 / 56, 103 / 99; 337 MiB 69 / 67, 115 / 107; 1580 MiB 322 / 292, 374 / 334; bf16 8 x 32,
// 195 MiB 33 / 35, 70 / 67; 292 MiB 54 / 52, 102 / 94; 341 MiB 71 / 67, 112 / 104; fp32 8 x 8, 230 MiB 36 / 38, 81 / 75; 345 MiB 69 / 65, 109 / 99.
// Once / resident by the bytes a wavefront moves at a time, least and most for arrays of 320 and 1500 MiB, cached and not:
//   856 to 1216  1.13 1.33  (bf16 2 x 100, 4 x 20, 5 x 40, 3 x 12, 4 x 12)        1264 to 1320  0.99 1.09  (2 x 36, 3 x 24)
//   1504         0.98 1.06  (4 x 20)             1628 to 1656  0.92 1.03  (1 x 200, 1 x 48, 2 x 100, 1 x 100)
//   1704         0.93 1.02  (3 x 32, bf16 3 x 64)       1860 0.86 0.99  (3 x 12)       2160 0.88 0.98  (4 x 64)       2816 0.83 0.87  (bf16 8 x 4)
//   unaligned, 280 and 1200 MiB: fp32 1 x 47 (1616) 0.97 1.12, bf16 (864) 1.29 1.34
int64_t begin_grid_most(int64_t n, const NodeGeo& geo, int g, int D)
{
    constexpr int64_t kOnce = 1 << 22;      // (a launch counts its threads in 32 bits)
    const int64_t heads = geo.hg.count(g), moved = heads * (2 * D * (int64_t)geo.hg.fb + 28);
    return !geo.ragged && geo.slots(g) * moved >= 1600 && n * moved > ((int64_t)336 << 20) ? kOnce : kMaxPersistentWGs;
}

#define SAR_DISPATCH_G(T, F, CALL)                                                   \
    switch (lanes_for((F), Vec<T>::N)) {                                             \
        case 4: { constexpr int kG = 4; CALL; } break;                                \
        case 8: { constexpr int kG = 8; CALL; } break;                                \
        case 16: { constexpr int kG = 16; CALL; } break;                              \
        case 32: { constexpr int kG = 32; CALL; } break;                              \
        default: { constexpr int kG = 64; CALL; } break;                              \
    }

f256::FwdP fwd_params(const FwdArgs& a)
{
    f256::FwdP p{};
    p.indptr = a.indptr; p.indices = a.indices; p.rows = a.rows;
    p.n_rows = a.n_rows; p.n_long = a.n_long; p.n_hub = a.n_hub;
    p.Z = a.Z; p.t = a.t; p.a_l = a.a_l; p.s = a.s; p.m = a.m; p.l = a.l; p.acc = a.acc; p.out = a.out; p.L = a.L;
    p.H = a.H; p.tag_shift = a.tag_shift; p.slope = a.slope; p.act = a.act;
    p.ld = a.ldz; p.ldh = a.ldh; p.D = a.D;
    return p;
}

f256::Tabs fwd_tabs(const PtrTab& zt, const PtrTab& tt)
{
    f256::Tabs tabs{};
    for (int q = 0; q < SAR_MAX_BLOCKS; ++q) {
        tabs.Z[q] = zt.p[q];
        tabs.t[q] = static_cast<const float*>(tt.p[q]);
    }
    return tabs;
}

constexpr int kHubWaves = 12;
// A call over all blocks.
template <typename T, int LPH, bool FLY, bool PAD, int NW>
int launch_fwd_waves(const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, hipStream_t st)
{
    constexpr int B = LPH >= 8 ? 8 : 4;
    auto fn = f256::k_gat_fwd_f256<T, LPH, B, FLY, PAD, NW>;
    // Formed scores of 4 or 8 heads and 1 KiB rows: registers let eight workgroups of four run on a CU, but seven are
    // faster (1 M rows of 2 edges, 4 heads of 64: 594 us with eight, 498 with seven; 100 thousand rows of 40, some of
    // them thousands long: 459 and 450).  The others lose by it (2 M edges to rows of bf16, given scores: 354 and 370).
    constexpr bool seven = NW == kWavesPerWG && FLY && !PAD && sizeof(T) == 4 && (LPH == 8 || LPH == 16);
    static const int resident = std::min(resident_workgroups(fn, NW * kWave), seven ? kMaxPersistentWGs / 8 * 7 : kMaxPersistentWGs);
    fn<<<persistent_grid_for(a.n_rows, a.n_long, resident, NW), NW * kWave, 0, st>>>(fwd_params(a), fwd_tabs(zt, tt));
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <typename T, int LPH, bool FLY, bool PAD>
int launch_fwd_f256(const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, hipStream_t st)
{
    return a.n_hub > 0 ? launch_fwd_waves<T, LPH, FLY, PAD, kHubWaves>(a, zt, tt, st)
                       : launch_fwd_waves<T, LPH, FLY, PAD, kWavesPerWG>(a, zt, tt, st);
}

template <typename T, int LPH, bool FLY, bool RAG>
int launch_fwd_slots(const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, int n_slots, hipStream_t st)
{
    auto fn = slots::k_gat_fwd_slots<T, LPH, FLY, RAG>;
    static const int resident = resident_workgroups(fn);
    fn<<<persistent_grid_for(a.n_rows, a.n_long, resident), kGatherThreads, 0, st>>>(fwd_params(a), fwd_tabs(zt, tt),
                                                                                     n_slots);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// A call over one block: the rows of 8 edges and more and the others in one launch.
template <typename T, int LPH, bool FLY, bool RAG, bool WHOLE, bool PAD>
int launch_fwd_block(const FwdArgs& a, hipStream_t st)
{
    auto fn = slots::k_gat_fwd_block<T, LPH, FLY, RAG, WHOLE, PAD>;
    static const int resident = resident_workgroups(fn);
    f256::FwdP p = fwd_params(a);
    p.n_rows = a.n_wide;
    p.n_long = std::min(a.n_long, a.n_wide);
    int n_slots = 1;
    while (n_slots * 2 * a.H * LPH <= kWave) n_slots *= 2;
    const int64_t few = a.n_rows - a.n_wide, per_wg = (int64_t)n_slots * kWavesPerWG;
    const unsigned g_wide = a.n_wide > 0 ? persistent_grid_for(p.n_rows, p.n_long, resident) : 0;
    const unsigned g_few = (unsigned)std::min<int64_t>((few + per_wg - 1) / per_wg, resident);
    fn<<<g_wide + g_few, kGatherThreads, 0, st>>>(p, n_slots, (int)g_wide, a.n_wide, a.n_rows);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// The generic kernels' launch.
template <typename T, bool ALL>
int launch_fwd_generic(const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, int P, hipStream_t st)
{
    const unsigned grid = persistent_grid(a.n_rows, a.n_long);
    if constexpr (ALL) {
        if (a.act == SAR_ACT_RELU) {
            SAR_DISPATCH_G(T, a.F, (k_gat_fwd<T, kG, true, true><<<grid, kGatherThreads, 0, st>>>(a, zt, tt, P)));
            SAR_LAUNCH_CHECK();
            return SAR_OK;
        }
    }
    SAR_DISPATCH_G(T, a.F, (k_gat_fwd<T, kG, ALL, false><<<grid, kGatherThreads, 0, st>>>(a, zt, tt, P)));
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

// Runs `...` with T bound to the generic kernels' row type: whole 16-byte pieces (bf16 heads of more
// than 256 values, and what the forward pass keeps there) or, below 4 values, one or two of them.
#define SAR_DISPATCH_GENERIC(dtype, D, ...)                             \
    do {                                                                \
        const int piece_ = piece_for((dtype) == SAR_F32, D);            \
        if ((dtype) == SAR_F32) {                                       \
            if (piece_ == 4) {                                          \
                using T = float;                                        \
                __VA_ARGS__;                                            \
            } else if (piece_ == 2) {                                   \
                using T = f32x2_t;                                      \
                __VA_ARGS__;                                            \
            } else {                                                    \
                using T = f32x1_t;                                      \
                __VA_ARGS__;                                            \
            }                                                           \
        } else if (piece_ == 8) {                                       \
            using T = bf16_t;                                           \
            __VA_ARGS__;                                                \
        } else if (piece_ == 4) {                                       \
            using T = bf16x4_t;                                         \
            __VA_ARGS__;                                                \
        } else if (piece_ == 2) {                                       \
            using T = bf16x2_t;                                         \
            __VA_ARGS__;                                                \
        } else {                                                        \
            using T = bf16x1_t;                                         \
            __VA_ARGS__;                                                \
        }                                                               \
    } while (0)

#define SAR_FWD_F256(LPH, PAD)                                                                                       \
    case LPH:                                                                                                        \
        if constexpr (ALL)                                                                                           \
            return a.a_l ? launch_fwd_f256<T, LPH, true, PAD>(a, zt, tt, st) : launch_fwd_f256<T, LPH, false, PAD>(a, zt, tt, st); \
        else                                                                                                         \
            return a.a_l ? launch_fwd_block<T, LPH, true, false, true, PAD>(a, st)                                   \
                         : launch_fwd_block<T, LPH, false, false, true, PAD>(a, st)
#define SAR_FWD_SLOTS(LPH, RAG)                                                                                      \
    case LPH:                                                                                                        \
        if constexpr (ALL)                                                                                           \
            return a.a_l ? launch_fwd_slots<T, LPH, true, RAG>(a, zt, tt, geo.n_slots, st)                           \
                         : launch_fwd_slots<T, LPH, false, RAG>(a, zt, tt, geo.n_slots, st);                         \
        else                                                                                                         \
            return a.a_l ? launch_fwd_block<T, LPH, true, RAG, false, false>(a, st)                                  \
                         : launch_fwd_block<T, LPH, false, RAG, false, false>(a, st)

template <typename T, bool ALL>
int launch_fwd_fast(const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, const LaunchGeo& geo, hipStream_t st)
{
    if (geo.kind == Gather::kExact) {
        switch (geo.lph) {
            SAR_FWD_F256(4, false);
            SAR_FWD_F256(8, false);
            SAR_FWD_F256(16, false);
            SAR_FWD_F256(32, false);
            SAR_FWD_F256(64, false);
            default: break;
        }
    } else if (geo.kind == Gather::kPadded) {
        switch (geo.lph) {
            SAR_FWD_F256(8, true);
            SAR_FWD_F256(16, true);
            SAR_FWD_F256(32, true);
            SAR_FWD_F256(64, true);
            default: break;
        }
    } else if (geo.ragged) {
        switch (geo.lph) {
            SAR_FWD_SLOTS(4, true);
            SAR_FWD_SLOTS(8, true);
            SAR_FWD_SLOTS(16, true);
            SAR_FWD_SLOTS(32, true);
            SAR_FWD_SLOTS(64, true);
            default: break;
        }
    } else {
        switch (geo.lph) {
            SAR_FWD_SLOTS(4, false);
            SAR_FWD_SLOTS(8, false);
            SAR_FWD_SLOTS(16, false);
            SAR_FWD_SLOTS(32, false);
            default: break;
        }
    }
    return sar::fail(SAR_ERR_STATE, "no forward kernel for %d heads of %d values", a.H, a.D);
}

template <bool ALL>
int launch_fwd(int dtype, const FwdArgs& a, const PtrTab& zt, const PtrTab& tt, int P, hipStream_t st)
{
    if (a.n_rows == 0) return SAR_OK;
    const LaunchGeo geo = launch_geo(dtype, a.H, a.D, a.ldz, fwd_pass(a.a_l == nullptr, ALL));
    if (geo.kind == Gather::kGeneric)
        SAR_DISPATCH_GENERIC(dtype, a.D, return (launch_fwd_generic<T, ALL>(a, zt, tt, P, st)));
    if (dtype == SAR_F32) return launch_fwd_fast<float, ALL>(a, zt, tt, geo, st);
    return launch_fwd_fast<bf16_t, ALL>(a, zt, tt, geo, st);
}

// Work of a backward launch in the padded geometry or with slots: kernels, and what they need
// besides BwdTabs and BwdP.
f256::BwdTabs bwd_tabs(const BwdArgs& tabs)
{
    f256::BwdTabs t{};
    for (int q = 0; q < SAR_MAX_BLOCKS; ++q) {
        t.t_indptr[q] = tabs.t_indptr[q]; t.t_indices[q] = tabs.t_indices[q];
        t.Z[q] = tabs.Z[q]; t.t[q] = tabs.t[q]; t.dZ[q] = tabs.dZ[q]; t.dt[q] = tabs.dt[q];
        t.rank[q] = tabs.rank[q];
    }
    return t;
}

f256::BwdP bwd_params(const BwdScalars& a)
{
    f256::BwdP p{};
    p.rows = a.rows; p.n_rows = a.n_wide; p.n_long = std::min(a.n_long, a.n_wide);
    p.G = a.G; p.rec = a.rec; p.a_l = a.a_l; p.ds = a.ds;
    p.ds_stride = a.ds_stride; p.ds_copies = a.ds_copies; p.partial = a.partial;
    p.H = a.H; p.tag_shift = a.tag_shift; p.slope = a.slope;
    p.ld = a.ldz; p.ldh = a.ldh; p.D = a.D;
    return p;
}

// Workgroups of the wide kernel.  Its fp32 form fills the memory's queues with two workgroups a CU (eight wavefronts with eight
// rows of 1 KiB each under way, 64 KiB; 7 TB/s over 2 us are 55), and more of them only push the frequent destinations' rows out
// of L2: 15 M edges, 4 x 64, 1577 us with five a CU, 1555 with three, 1508 with two; 122 M edges, 4 x 100, 36.4, 36.3
// and 36.1 ms.  Launches in which a wavefront has few sources want them all the same (4 x 64 over 0.7 M edges 38 us, with two a
// CU 41; 2 x 100 over 1 M 66 and 71), and so do bf16 rows (201 M edges 5.4 and 5.7 ms; 8 M 611 and 795 us), and shorter
// rows, of which two workgroups have too little under way.  (The call, two a CU / all, two power-law and two uniform graphs of 8 to 21 M
// edges, by bytes of a row in a launch: 432, 6 x 36, 1.04 to 1.07; 480 and 320, 5 x 40, 1.02 to 1.03; 576, 3 x 48 and 4 x 36, 0.97 to 1.04;
// 640, 4 x 40, 1.00 to 1.04; 640 and 320, 3 x 80, 0.98 to 1.00; 672, 3 x 56, 0.95 to 1.00; 704 to 736, 0.95 to 1.01; 768, 1 x 192 to
// 4 x 48, 0.94 to 1.03, six of sixteen up to 0.99 and two above 1.01; 896, 4 x 56, 0.97 to 0.99; 1024, 0.98 to 0.99, and 16 x 16, with
// four rows under way, 0.99 to 1.01.)
template <typename T>
unsigned wide_grid(const f256::BwdP& p, int resident)
{
    constexpr int kTwoPerCu = kMaxPersistentWGs / 4, kShort = 640;
    const bool many = sizeof(T) == 4 && p.H * p.D * (int)sizeof(T) > kShort &&
                      p.n_rows >= (int64_t)kTwoPerCu * kWavesPerWG * kWave;
    return persistent_grid_for(p.n_rows, p.n_long, many ? std::min(resident, kTwoPerCu) : resident);
}

// The padded and the slots kernels.  The few-edges kernels also take the sources without an edge
// at the end of the list (they write their zero rows).
template <typename T, int LPH, bool ALL, bool SLOTS, bool RAG>
int launch_bwd_padded(const BwdArgs& tabs, const BwdScalars& a, int n_slots, unsigned* grid_out, hipStream_t st)
{
    constexpr int B = LPH >= 8 ? 8 : 4;
    const f256::BwdTabs t = bwd_tabs(tabs);
    const f256::BwdP p = bwd_params(a);
    unsigned g_wide = 0, g_few = 0, g_single = 0;
    // The sources of one edge go destination-major where the handle lists them that way.  In the
    // work list they sit between the other few-edge sources and the ones without an edge, so the
    // few-edges part takes the list in two pieces around them.
    const int64_t n_edged = std::max(a.n_wide, std::min(a.n_rows, a.n_touched));
    const int64_t n_pulled = (!RAG && ALL && a.s_dst && a.n_single <= n_edged - a.n_wide) ? a.n_single : 0;
    const int64_t piece[2][2] = {{a.n_wide, n_pulled ? n_edged - n_pulled : a.n_rows}, {n_edged, n_pulled ? a.n_rows : n_edged}};
    if (!a.wide_done && (!SLOTS || n_pulled > 0)) {       // (the slots kernel takes both kinds of sources as it is)
        constexpr joint::Lanes lanes = SLOTS ? joint::Lanes::kSlots : joint::Lanes::kPadded;
        const joint::Work w{{{piece[0][0], piece[0][1]}, {piece[1][0], piece[1][1]}}, {a.s_dst, a.s_src, a.s_row, n_pulled, 0},
                            n_slots, LPH, lanes, ALL};
        int grid = 0;
        SAR_TRY(sar::bwd_joint(sizeof(T) == 4 ? SAR_F32 : SAR_BF16, t, p, w, &grid, st));
        *grid_out = (unsigned)grid;
        if (grid > 0) return SAR_OK;
    }
    if constexpr (SLOTS) {
        auto kernel = slots::k_gat_bwd_slots<T, LPH, ALL, RAG>;
        static const int resident = resident_workgroups(kernel);
        if (a.n_wide > 0 && !a.wide_done) g_wide = persistent_grid_for(p.n_rows, p.n_long, resident);
        for (int k = 0; k < 2; ++k) {
            const int64_t n = piece[k][1] - piece[k][0];
            const unsigned wide = k == 0 ? g_wide : 0;
            const unsigned g = n > 0 ? grid_of(n, (int64_t)n_slots * kWavesPerWG, resident) : 0;
            if (wide + g == 0) continue;
            kernel<<<wide + g, kGatherThreads, 0, st>>>(t, p, n_slots, (int)wide, piece[k][0], piece[k][1],
                                                        (int)(k == 0 ? 0 : g_wide + g_few));
            SAR_LAUNCH_CHECK();
            g_few += g;
        }
    } else {
        auto wide = f256::k_gat_bwd_f256<T, LPH, B, ALL, true>;
        auto few = f256::k_gat_bwd_few<T, LPH, ALL, true>;
        static const int resident_wide = resident_workgroups(wide), resident_few = resident_workgroups(few);
        if (a.n_wide > 0 && !a.wide_done) {
            g_wide = wide_grid<T>(p, resident_wide);
            wide<<<g_wide, kGatherThreads, 0, st>>>(t, p);
            SAR_LAUNCH_CHECK();
        }
        for (int k = 0; k < 2; ++k) {
            const int64_t n = piece[k][1] - piece[k][0];
            if (n <= 0) continue;
            const unsigned g = grid_of(n, (int64_t)(B / 2) * kWavesPerWG, resident_few);
            few<<<g, kGatherThreads, 0, st>>>(t, p, piece[k][0], piece[k][1], (int)(g_wide + g_few));
            SAR_LAUNCH_CHECK();
            g_few += g;
        }
    }
    if constexpr (!RAG && ALL) {
        if (n_pulled > 0) {
            auto single = f256::k_gat_bwd_single<T, LPH, true>;
            static const int resident = resident_workgroups(single);
            const f256::SingleP sp = single_list({a.s_dst, a.s_src, a.s_row, n_pulled, 0}, resident, g_single);
            single<<<g_single, kGatherThreads, 0, st>>>(t, p, sp, (int)(g_wide + g_few));
            SAR_LAUNCH_CHECK();
        }
    }
    *grid_out = g_wide + g_few + g_single;
    return SAR_OK;
}

// da_l[h*D + off(k) + x] += sum_w partial[w][(h*LPH + k)*4 + x]: the padded and the slots kernels
// leave their partial sums in lane order (256 per workgroup).  off(k) = 4k, or D - 4 for the last
// lane of a ragged head; the values such a lane shares with the one before it are that one's.
template <int COLS>
__global__ __launch_bounds__(256) void k_reduce_partials_padded(const float* __restrict__ partial, int n_part,
                                                                int lph, int H, int D, float* __restrict__ out)
{
    const int slot = blockIdx.x * COLS, lane = slot / 4, h = lane / lph, k = lane % lph, off = min(4 * k, D - 4);
    if (h >= H || 4 * k >= D) return;
    add_columns<COLS>(partial + slot, n_part, 256, [&](int c) -> float* {
        const int x = slot % 4 + c;
        return off + x < 4 * k ? nullptr : out + h * D + off + x;
    });
}

// The sources without an edge in their block (the tail of the work list): their rows of dZ_q and
// dt_q are zero, and nothing has to be read for that but the list entry.
template <typename T, bool ALL>
__global__ __launch_bounds__(256) void k_bwd_zero_rows(f256::BwdTabs tabs, const uint32_t* __restrict__ rows,
                                                       int64_t r_begin, int64_t r_end, int H, int tag_shift)
{
    constexpr int kPieces = f256::kF * (int)sizeof(T) / 16;   // 16-byte pieces of a row
    __shared__ GlobalPtr<void> s_dZ[SAR_MAX_BLOCKS];
    __shared__ GlobalPtr<float> s_dt[SAR_MAX_BLOCKS];
    if (threadIdx.x < SAR_MAX_BLOCKS) {
        s_dZ[threadIdx.x] = tabs.dZ[threadIdx.x];
        s_dt[threadIdx.x] = tabs.dt[threadIdx.x];
    }
    __syncthreads();
    const uint32_t mask = ALL ? ((1u << tag_shift) - 1u) : 0xffffffffu;
    const int64_t total = (r_end - r_begin) * kPieces;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < total; p += (int64_t)gridDim.x * 256) {
        const uint32_t id = rows[r_begin + p / kPieces];
        const int piece = (int)(p % kPieces);
        const int q = ALL ? (int)(id >> tag_shift) : 0;
        const int64_t j = (int64_t)(id & mask);
        reinterpret_cast<uint4*>(s_dZ[q].template as<T>() + j * f256::kF)[piece] = make_uint4(0u, 0u, 0u, 0u);
        if (piece < H && s_dt[q]) s_dt[q][j * H + piece] = 0.f;
    }
}

__global__ __launch_bounds__(256) void k_zero_f32(float* __restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0.f;
}

template <typename T, int LPH, bool ALL>
int launch_bwd_f256(const BwdArgs& tabs, const BwdScalars& a, unsigned* grid_out, hipStream_t st)
{
    constexpr int B = LPH >= 8 ? 8 : 4;
    auto wide = f256::k_gat_bwd_f256<T, LPH, B, ALL, false>;
    auto few = f256::k_gat_bwd_few<T, LPH, ALL, false>;
    auto single = f256::k_gat_bwd_single<T, LPH, false>;
    constexpr int kPerWave = B / 2;     // sources a wavefront of that kernel takes at once
    static const int resident_wide = resident_workgroups(wide);
    static const int resident_few = resident_workgroups(few);
    static const int resident_single = resident_workgroups(single);
    const f256::BwdTabs t = bwd_tabs(tabs);
    const f256::BwdP p = bwd_params(a);
    unsigned g_wide = 0, g_few = 0, g_single = 0;
    const int64_t n_edged = std::max(a.n_wide, std::min(a.n_rows, a.n_touched));
    // the sources of one edge (the end of the edged part of the list) go destination-major where
    // the handle lists them that way
    const int64_t n_pulled = (ALL && a.s_dst && a.n_single <= n_edged - a.n_wide) ? a.n_single : 0;
    const int64_t n_few_end = n_edged - n_pulled;
    // Where many sources have no edge (a 16-way split leaves 46% of them without one), their 32-byte
    // rows of dt_q scattered through the array cost more to zero one by one than the whole array
    // does in one sweep ahead of the kernels that write the other rows.
    const bool sweep_dt = a.n_src_host != nullptr && (a.n_rows - n_edged) * 4 > a.n_rows;
    if (sweep_dt) {
        for (int q = 0; q < a.n_blocks; ++q) {
            const int64_t n = a.n_src_host[q] * a.H;
            if (n == 0 || !tabs.dt[q]) continue;
            k_zero_f32<<<(unsigned)std::min<int64_t>((n + 255) / 256, kMaxPersistentWGs), 256, 0, st>>>(tabs.dt[q], n);
            SAR_LAUNCH_CHECK();
        }
    }
    int g_joint = 0;
    if (!a.wide_done) {
        const joint::Work w{{{a.n_wide, n_few_end}, {0, 0}}, {a.s_dst, a.s_src, a.s_row, n_pulled, 0}, 1, LPH,
                            joint::Lanes::kExact, ALL};
        SAR_TRY(sar::bwd_joint(sizeof(T) == 4 ? SAR_F32 : SAR_BF16, t, p, w, &g_joint, st));
    }
    if (g_joint == 0 && a.n_wide > 0 && !a.wide_done) {
        // sources with at least 8 edges: one wavefront (or workgroup) each
        g_wide = wide_grid<T>(p, resident_wide);
        wide<<<g_wide, kGatherThreads, 0, st>>>(t, p);
        SAR_LAUNCH_CHECK();
    }
    if (g_joint == 0 && n_few_end > a.n_wide) {
        // the other sources with edges, several per wavefront
        const int64_t n = n_few_end - a.n_wide;
        const int64_t per_wg = (int64_t)kPerWave * kWavesPerWG;
        g_few = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + per_wg - 1) / per_wg, resident_few));
        few<<<g_few, kGatherThreads, 0, st>>>(t, p, a.n_wide, n_few_end, (int)g_wide);
        SAR_LAUNCH_CHECK();
    }
    if (g_joint == 0 && n_pulled > 0) {
        const f256::SingleP sp = single_list({a.s_dst, a.s_src, a.s_row, n_pulled, 0}, resident_single, g_single);
        single<<<g_single, kGatherThreads, 0, st>>>(t, p, sp, (int)(g_wide + g_few));
        SAR_LAUNCH_CHECK();
    }
    if (a.n_rows > n_edged) {
        const int64_t pieces = (a.n_rows - n_edged) * (f256::kF * (int64_t)sizeof(T) / 16);
        const unsigned g_zero = (unsigned)std::min<int64_t>((pieces + 255) / 256, kMaxPersistentWGs);
        k_bwd_zero_rows<T, ALL><<<g_zero, 256, 0, st>>>(t, a.rows, n_edged, a.n_rows, sweep_dt ? 0 : a.H,
                                                       a.tag_shift);
        SAR_LAUNCH_CHECK();
    }
    *grid_out = g_joint + g_wide + g_few + g_single;
    return SAR_OK;
}

#define SAR_BWD_CASE(LPH, SLOTS, RAG)                                                                     \
    case LPH: SAR_TRY((launch_bwd_padded<T, LPH, ALL, SLOTS, RAG>(tabs, a, geo.n_slots, &grid, st))); break

template <typename T, bool ALL>
int launch_bwd_fast(const BwdArgs& tabs, const BwdScalars& a, const LaunchGeo& geo, float* da_l, hipStream_t st)
{
    unsigned grid = 0;
    if (geo.kind == Gather::kExact) {
        switch (geo.lph) {
            case 4: SAR_TRY((launch_bwd_f256<T, 4, ALL>(tabs, a, &grid, st))); break;
            case 8: SAR_TRY((launch_bwd_f256<T, 8, ALL>(tabs, a, &grid, st))); break;
            case 16: SAR_TRY((launch_bwd_f256<T, 16, ALL>(tabs, a, &grid, st))); break;
            case 32: SAR_TRY((launch_bwd_f256<T, 32, ALL>(tabs, a, &grid, st))); break;
            default: SAR_TRY((launch_bwd_f256<T, 64, ALL>(tabs, a, &grid, st))); break;
        }
        return reduce_partials(a.partial, (int)grid, a.F, da_l, st);
    }
    if (geo.kind == Gather::kPadded) {
        switch (geo.lph) {
            SAR_BWD_CASE(8, false, false);
            SAR_BWD_CASE(16, false, false);
            SAR_BWD_CASE(32, false, false);
            SAR_BWD_CASE(64, false, false);
            default: return sar::fail(SAR_ERR_STATE, "no backward kernel for %d heads of %d values", a.H, a.D);
        }
    } else if (geo.ragged) {
        switch (geo.lph) {
            SAR_BWD_CASE(4, true, true);
            SAR_BWD_CASE(8, true, true);
            SAR_BWD_CASE(16, true, true);
            SAR_BWD_CASE(32, true, true);
            SAR_BWD_CASE(64, true, true);
            default: return sar::fail(SAR_ERR_STATE, "no backward kernel for %d heads of %d values", a.H, a.D);
        }
    } else {
        switch (geo.lph) {
            SAR_BWD_CASE(4, true, false);
            SAR_BWD_CASE(8, true, false);
            SAR_BWD_CASE(16, true, false);
            SAR_BWD_CASE(32, true, false);
            default: return sar::fail(SAR_ERR_STATE, "no backward kernel for %d heads of %d values", a.H, a.D);
        }
    }
    if ((int)grid <= kFewPartials)
        k_reduce_partials_padded<4><<<256 / 4, 256, 0, st>>>(a.partial, (int)grid, geo.lph, a.H, a.D, da_l);
    else
        k_reduce_partials_padded<1><<<256, 256, 0, st>>>(a.partial, (int)grid, geo.lph, a.H, a.D, da_l);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <typename T, bool ALL>
int launch_bwd_generic(const BwdArgs& tabs, const BwdScalars& a, float* da_l, hipStream_t st)
{
    const unsigned grid = persistent_grid(a.n_rows, a.n_long);
    SAR_DISPATCH_G(T, a.F, (k_gat_bwd<T, kG, ALL><<<grid, kGatherThreads, 0, st>>>(tabs, a)));
    SAR_LAUNCH_CHECK();
    return reduce_partials(a.partial, (int)grid, a.F, da_l, st);
}

// The generic backward kernel's row types: heads of 1 to 3 values, bf16 heads of more than 256.
#define SAR_DISPATCH_GENERIC_BWD(dtype, D, ...)          \
    do {                                                 \
        if ((dtype) == SAR_F32) {                        \
            if ((D) == 2) {                              \
                using T = f32x2_t;                       \
                __VA_ARGS__;                             \
            } else {                                     \
                using T = f32x1_t;                       \
                __VA_ARGS__;                             \
            }                                            \
        } else if ((D) > 256) {                          \
            using T = bf16_t;                            \
            __VA_ARGS__;                                 \
        } else if ((D) == 2) {                           \
            using T = bf16x2_t;                          \
            __VA_ARGS__;                                 \
        } else {                                         \
            using T = bf16x1_t;                          \
            __VA_ARGS__;                                 \
        }                                                \
    } while (0)

template <bool ALL>
int launch_bwd(int dtype, const BwdArgs& tabs, const BwdScalars& a, float* da_l, hipStream_t st)
{
    if (a.n_rows == 0) return SAR_OK;
    const LaunchGeo geo = launch_geo(dtype, a.H, a.D, a.ldz, Pass::kBwd);
    if (geo.kind == Gather::kGeneric)
        SAR_DISPATCH_GENERIC_BWD(dtype, a.D, return (launch_bwd_generic<T, ALL>(tabs, a, da_l, st)));
    if (dtype == SAR_F32) return launch_bwd_fast<float, ALL>(tabs, a, geo, da_l, st);
    return launch_bwd_fast<bf16_t, ALL>(tabs, a, geo, da_l, st);
}

// room for one row of 256 partial sums per workgroup of the (up to) four backward launches of a call
size_t workspace_bytes(int F) { return (size_t)4 * kMaxPersistentWGs * F * sizeof(float); }

// The backward kernels add every edge's du to ds with atomics.  ds is small (4H bytes a destination),
// so the frequent destinations of a power-law graph share few cache lines (32/H of them a line), and
// additions to one line are served one after the other, some 4 ns each: on a share of 7.4M edges and
// 150k destinations, 1 x 47, the two backward kernels took 1019 + 688 us with and 255 + 183 us without
// the additions.  Where that is what a call would wait for, the workgroups add to several copies of ds
// (copy = workgroup modulo their number, so with 8 or more an XCD's workgroups have theirs to
// themselves), summed at the end: 399 + 250 us with 8 copies, 344 + 231 with 16; bf16 4 x 64 on 31k
// destinations 230 + 293 -> 72 + 91.  Copies are kept small (up to 1.25 MB 16 of them, to 2.5 MB 8:
// zeroing and summing them is 10 to 15 us): ds of 4.9 MB (4 x 64 on 306k destinations) is spread
// over enough lines, 1530 + 1324 us as it is and 1535 + 1364 with 8 copies.
constexpr size_t kDsSmall = 5 << 18;
int ds_copies_for(int64_t n_dst, int H)
{
    const size_t bytes = (size_t)n_dst * H * sizeof(float);
    return bytes == 0 || bytes > 2 * kDsSmall ? 1 : bytes > kDsSmall ? 8 : 16;
}
// Whether a call of nnz edges to n_dst destinations, hub of them to the most frequent one, waits for ds: the additions to the
// line that destination is on, as if the line's other destinations were as frequent; or where the lines are few, those to every
// line, some 16 ns each there (262 destinations of 290 edges, 4 heads: 2300 a line and launch, the wide kernel 45 us without
// copies and 15 with).
// Copies are two more launches, 5 us of a small ds and 12 of 2.5 MB.  Steps of 3700 layers over power-law and uniform
// graphs (77 to 160 thousand destinations, 1 to 16 blocks, fourteen shapes): 11% longer than with the better of the two where
// copies are never taken, 1.8% always, 1.1% by the first line drawn at 20 us alone, 0.5% by both; worst 3.1, 1.11, 1.8 and
// 1.19 times.  Block by block, 712 layers: 2.8, 10.5, 1.1, 0.5%.
bool ds_contended(int64_t hub, int64_t nnz, int64_t n_dst, int H, int D, size_t fb)
{
    const double line_us = 0.004 * (double)hub * std::max(1, 32 / H);
    const double rows_us = (double)nnz * H * D * fb / 6e6;
    const double to_a_line = (double)nnz / std::max(1.0, (double)n_dst * H * sizeof(float) / 128.0);
    return (line_us > 10.0 && line_us > 0.05 * rows_us) || (to_a_line > 800.0 && 0.016 * to_a_line > 0.3 * rows_us);
}
size_t ds_copy_bytes(int64_t n_dst, int H) { return ((size_t)n_dst * H * sizeof(float) + 255) / 256 * 256; }

// ds[i] += sum of the copies' ds[i] (COPIES = 8 or 16: their loads travel together)
template <int COPIES>
__global__ __launch_bounds__(256) void k_ds_sum(const float* __restrict__ copies, int64_t stride,
                                                float* __restrict__ ds, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        float v[COPIES], s = 0.f;
#pragma unroll
        for (int c = 0; c < COPIES; ++c) v[c] = copies[c * stride + i];
#pragma unroll
        for (int c = 0; c < COPIES; ++c) s += v[c];
        ds[i] += s;
    }
}

// Scratch of a backward pass by head slices, behind the copies of ds: a record and a ds of every destination and head.
// None is set aside for more than 2^20 of these, 20 MiB for every caller whatever its graph: beyond, with 8 heads, a graph
// has 34 million edges and more where slices are taken (two uses: n_dst^2 / 512 edges).  By rows / by slices there, us: 160
// thousand destinations, 8 x 32, 64 M edges 10060 / 10240; 200 thousand, 100 M 15770 / 14250; 280 thousand, 4 x 64, 168 M
// 26750 / 25370.
size_t slices_bytes(int64_t n_dst, int H)
{
    return n_dst * H <= (int64_t)1 << 20 ? (size_t)n_dst * H * 5 * sizeof(float) : 0;
}

// Where a backward call's atomics go: ds itself or zeroed copies of it in the caller's scratch.
struct DsTarget {
    float* base;
    int64_t stride, n;
    int copies;
};
int ds_begin(DsTarget& d, int64_t n_dst, bool contended, int H, float* ds, void* work, size_t work_bytes, hipStream_t st)
{
    d = DsTarget{ds, 0, n_dst * H, 1};
    const int c = ds_copies_for(n_dst, H);
    const size_t each = ds_copy_bytes(n_dst, H);
    if (c == 1 || !contended || work_bytes < workspace_bytes(256) + c * each) return SAR_OK;
    d.base = reinterpret_cast<float*>(static_cast<char*>(work) + workspace_bytes(256));
    d.stride = (int64_t)(each / sizeof(float));
    d.copies = c;
    const int64_t n = d.stride * c;
    k_zero_f32<<<(unsigned)std::min<int64_t>((n + 255) / 256, kMaxPersistentWGs), 256, 0, st>>>(d.base, n);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}
int ds_end(const DsTarget& d, float* ds, hipStream_t st)
{
    if (d.copies == 1) return SAR_OK;
    const unsigned grid = (unsigned)std::min<int64_t>((d.n + 255) / 256, kMaxPersistentWGs);
    if (d.copies == 16)
        k_ds_sum<16><<<grid, 256, 0, st>>>(d.base, d.stride, ds, d.n);
    else
        k_ds_sum<8><<<grid, 256, 0, st>>>(d.base, d.stride, ds, d.n);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

}  // namespace

// One pass over Z for one or two score vectors (a2/score2 may be null).
int sar::gat_scores2(const void* Z, int dtype, int64_t n, int H, int D, const float* a, float* score,
                     const float* a2, float* score2, void* stream)
{
    if (dtype != SAR_F32 && dtype != SAR_BF16)
        return sar::fail(SAR_ERR_UNSUPPORTED, "dtype %d is neither SAR_F32 nor SAR_BF16", dtype);
    SAR_CHECK_ARG(H > 0 && D > 0, "H and D must be positive (H=%d, D=%d)", H, D);
    SAR_CHECK_ARG((a2 == nullptr) == (score2 == nullptr), "the second vector and its output go together");
    if (D / piece_for(dtype == SAR_F32, D) > 64) {
        // a head that no wavefront covers in lane pieces (an odd width above 64, say): one thread
        // per (node, head); any width is a valid product of the transform
        SAR_CHECK_ARG(n >= 0, "n is negative");
        if (n == 0) return SAR_OK;
        SAR_CHECK_ARG(Z && a && score, "Z, a or score is null");
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n * H + 255) / 256, kMaxPersistentWGs * 4));
        if (dtype == SAR_F32)
            k_scores_any<float><<<grid, 256, 0, sar::as_stream(stream)>>>(static_cast<const float*>(Z), n, H, D, a,
                                                                          score, a2, score2);
        else
            k_scores_any<bf16_t><<<grid, 256, 0, sar::as_stream(stream)>>>(static_cast<const bf16_t*>(Z), n, H, D, a,
                                                                           score, a2, score2);
        SAR_LAUNCH_CHECK();
        return SAR_OK;
    }
    SAR_TRY(check_shape(dtype, H, D));
    SAR_CHECK_ARG(n >= 0, "n is negative");
    if (n == 0) return SAR_OK;
    SAR_CHECK_ARG(Z && a && score, "Z, a or score is null");
    SAR_CHECK_ARG(aligned16(Z), "Z must be 16-byte aligned");
    const NodeGeo geo = node_geo(dtype, H, D);
    hipStream_t st = sar::as_stream(stream);
    for (int g = 0; g < geo.hg.n; ++g) {
        const size_t h0 = (size_t)geo.hg.first(g), f0 = h0 * D;
        const void* Zg = shift(Z, f0 * geo.hg.fb);
        const unsigned grid = nodewise_grid(n, geo.slots(g));
        SAR_DISPATCH_NODE(dtype, geo, (k_scores<T, kV, kL, kR><<<grid, kGatherThreads, 0, st>>>(
                                          static_cast<const T*>(Zg), n, geo.hg.count(g), D, H * D, H, a + f0, score + h0,
                                          a2 ? a2 + f0 : nullptr, score2 ? score2 + h0 : nullptr)));
        SAR_LAUNCH_CHECK();
    }
    return SAR_OK;
}

extern "C" int sar_gat_scores(const void* Z, int dtype, int64_t n, int H, int D, const float* a,
                              float* score, void* stream)
{
    return sar::gat_scores2(Z, dtype, n, H, D, a, score, nullptr, nullptr, stream);
}

extern "C" int sar_gat_fwd_begin(float* m, float* l, float* acc, int64_t n_dst, int H, int D, void* stream)
{
    SAR_CHECK_ARG(n_dst >= 0 && H > 0 && D > 0, "need n_dst >= 0, H > 0, D > 0");
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(m && l && acc, "m, l or acc is null");
    const int64_t n_f = n_dst * H * D;
    const unsigned grid = (unsigned)std::min<int64_t>((n_f + 255) / 256, 1 << 20);
    k_fwd_begin<<<grid, 256, 0, sar::as_stream(stream)>>>(m, l, acc, n_dst * H, n_f);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

extern "C" int sar_gat_fwd_block(const sar_blocks_t* b, int q, const void* Zq, const float* s,
                                 const float* tq, const float* a_l, int dtype, int H, int D, float slope,
                                 float* m, float* l, float* acc, void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_CHECK_ARG(q >= 0 && q < b->P, "block %d out of range [0,%d)", q, b->P);
    SAR_TRY(check_shape(dtype, H, D));
    const sar::Block& k = b->blk[q];
    if (k.n_rows == 0) return SAR_OK;
    SAR_CHECK_ARG(Zq && s && m && l && acc, "a tensor argument is null");
    SAR_CHECK_ARG(tq || a_l, "either tq or a_l must be given");
    SAR_CHECK_ARG(aligned16(Zq) && aligned16(acc) && aligned16(a_l), "Zq, acc and a_l must be 16-byte aligned");
    const HeadGroups hg = head_groups(dtype, H, D, fwd_pass(tq != nullptr, false));
    for (int g = 0; g < hg.n; ++g) {
        const size_t h0 = (size_t)hg.first(g), f0 = h0 * D;
        FwdArgs a{};
        a.indptr = k.indptr;
        a.indices = reinterpret_cast<const uint32_t*>(k.indices);
        a.rows = reinterpret_cast<const uint32_t*>(k.rows);
        a.n_rows = k.n_rows;
        a.n_long = k.n_shared;
        a.n_wide = k.n_rows_wide;
        a.Z = shift(Zq, f0 * hg.fb);
        a.t = tq ? tq + h0 : nullptr;
        a.a_l = tq ? nullptr : a_l + f0;
        a.s = s + h0;
        a.m = m + h0;
        a.l = l + h0;
        a.acc = acc + f0;
        a.H = hg.count(g);
        a.D = D;
        a.F = a.H * D;
        a.ldz = H * D;
        a.ldh = H;
        a.slope = slope;
        PtrTab none{};
        SAR_TRY(launch_fwd<false>(dtype, a, none, none, 0, sar::as_stream(stream)));
    }
    return SAR_OK;
}

extern "C" int sar_gat_fwd_end(const float* m, const float* l, const float* acc, int act, void* out, float* L,
                               int dtype, int64_t n_dst, int H, int D, void* stream)
{
    SAR_TRY(check_shape(dtype, H, D));
    SAR_TRY(check_act(act));
    SAR_CHECK_ARG(n_dst >= 0, "n_dst is negative");
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(m && l && acc && out && L, "a tensor argument is null");
    SAR_CHECK_ARG(aligned16(acc) && aligned16(out), "acc and out must be 16-byte aligned");
    const NodeGeo geo = node_geo(dtype, H, D);
    hipStream_t st = sar::as_stream(stream);
    for (int g = 0; g < geo.hg.n; ++g) {
        const size_t h0 = (size_t)geo.hg.first(g), f0 = h0 * D;
        const unsigned grid = nodewise_grid(n_dst, geo.slots(g));
        SAR_DISPATCH_NODE(dtype, geo, (k_fwd_end<T, kV, kL, kR><<<grid, kGatherThreads, 0, st>>>(
                                          m + h0, l + h0, acc + f0, static_cast<T*>(out) + f0, L + h0, n_dst,
                                          geo.hg.count(g), D, H * D, H, act)));
        SAR_LAUNCH_CHECK();
    }
    return SAR_OK;
}

namespace {

// Which passes over all blocks go by head slices (gat_slices.h).
//
// An XCD walks 512 wavefronts' rows together and fetches the slices of the table that these cite once per such sweep:
// `uses` is how often it then uses a fetched slice (rows of `edges` edges together gathering from a table of `table` rows,
// `sets` slices to a row of the table, `lanes` lanes to a slice).  It pays from two uses on, and where there are at least
// four sweeps: with fewer the chip is not full (8 thousand nodes, 2 x 100, 100 edges a row, two sweeps: 54 us forward by
// rows, 74 by slices; 10 thousand, 4 x 64, 50 edges: 61 / 100 backward).  No row may be far longer than the others: a
// lane group walks it alone while the workgroup waits.
bool even_rows(int64_t rows, int64_t edges, int64_t longest)
{
    return rows > 0 && edges > 0 && longest > 0 && longest * rows <= 4 * edges;
}
bool sets_for_xcds(int sets) { return sets == 1 || sets == 2 || sets == 4 || sets % slices::kXcds == 0; }
bool sweeps_pay(int sets, int lanes, int64_t rows, int64_t edges, int64_t table, double least_uses)
{
    const int parts = sets < slices::kXcds ? slices::kXcds / sets : 1;
    const double sweeps = rows / (parts * 512.0 * (kWave / lanes)), uses = edges / (parts * std::max(sweeps, 1.0) * table);
    return sweeps >= 4.0 && uses >= least_uses;
}

// Forward over all blocks by rows: how many rows at the head of the list all twelve wavefronts of a workgroup share (0:
// workgroups of four).  A workgroup of four takes 32 edges of a row per round trip to memory, so a row of more edges than
// its fair share (about 2048 of them run at once) decides when the launch ends.  Workgroups of twelve hold 24 wavefronts on a
// CU instead of 32, and a row of a few times their 768 edges is soon over either way.  Times of twelve over four in turn on
// 2600 shares of power-law graphs (20 thousand to 16 million edges, 2 to 100 a row, twelve layers), where the longest row has
// at least a share:
//   - 4096 edges and more: 0.82 in the mean, 0.96 at the 90th percentile, 1.05 at most (1.5 M edges, rows up to 10143, 4 x 64
//     fp32 501 -> 358 us, bf16 434 -> 253; 9 M edges, 8 x 32 bf16 with given scores 1162 -> 1029);
//   - 2048 to 4095 (the class is what is known): 0.95; with 96 such rows of 1024 edges and more and a share and a half 0.9, 1.13
//     at most;
//   - 1024 to 2047: 1.08 to 1.41, most on small graphs (0.2 M edges 84 -> 114 us);
//   - rows of 1 KiB with scores formed in flight (4 x 64, 2 x 128 fp32): 1.00 up to two shares (15 M edges 2186 / 2181 and 2155
//     / 2184 us), 0.87 to 0.96 beyond.
// Less than a share: 1.02.  The forms for padded layers spill a few registers at twelve wavefronts (20 to 32 bytes a lane) and
// are among these figures; one workgroup of them per CU and no spills took 1.02 to 1.39 times as long as four wavefronts
// where this takes 0.92 to 0.99.
int64_t shared_hubs(const sar_blocks_t* b, size_t row_bytes, bool scores_given)
{
    const int64_t longest = (b->f_longest + 1) / 2;      // at least
    if (longest < 2048 || (longest < 4096 && b->n_f_hub < 96)) return 0;
    int64_t edges = 0;
    for (int q = 0; q < b->P; ++q) edges += b->blk[q].nnz;
    const double least = row_bytes >= 1024 && !scores_given ? 2.0 : longest < 4096 ? 1.5 : 1.0;
    return (double)longest * kMaxPersistentWGs >= least * (double)edges ? b->n_f_hub : 0;
}

// Forward: heads of 32 to 128 fp32 values or 64 to 128 bf16 values (slices of 128 bytes, a cache line, and more: 64-byte
// slices bring the neighbour's half along, 4 x 16 fp32 310 -> 440 us).  Tables that mostly stay in the L2s anyway gain
// nothing, and `whole`, the bytes of all sources' rows, says which.  Times of slices over rows on 7600 uniform graphs (6 to
// 370 thousand nodes, 16 to 500 edges a row, 1 to 16 blocks, 13 layers; mean, 90th percentile, most):
//   - the head's slices of the whole table within 3 of an XCD's 4 MiB of L2 and at least 10 thousand wavefronts of work:
//     no barriers.  fp32 from 12 MiB on 0.70, 0.83, 0.92 (20 thousand nodes, 8 x 32, 100 edges a row 215 -> 134 us), 8 to 12
//     MiB 0.8, 1.1, 1.2; bf16 1.05, 1.09, 1.27;
//   - else where sweeps pay.  fp32 from 20 MiB on 0.71, 0.89, 1.12 (50 thousand destinations of 200 thousand nodes, 8 x 32,
//     500 edges 3380 -> 2170 us, 100 edges, two uses, 700 -> 654), 12 to 20 MiB 0.9, 1.26, 1.5.  bf16 of one head 0.7, 0.8,
//     0.8; of several from 96 MiB on 0.93, 0.98, 0.98, 48 to 96 MiB 1.02, 1.1, 1.2, less 1.1 to 1.6;
//   - scores given, whose gathers cost each head a line more: fp32 from 24 MiB on 0.75, 0.90, 1.13, bf16 from 16 MiB on 0.84,
//     1.01, 1.25.  Where all eight XCDs gather another head's (8 heads and more) from five uses on; with two to three they
//     take 1.13 (12 M edges, 150 thousand nodes 1840 -> 2430 us).
enum class Slices { kNo, kFree, kSwept };
Slices fwd_by_slices(const sar_blocks_t* b, int dtype, int H, int D, bool scores_given)
{
    if (D % 4 != 0 || D > 128 || D < (dtype == SAR_F32 ? 32 : 64) || !sets_for_xcds(H)) return Slices::kNo;
    int64_t edges = 0, sources = 0;
    for (int q = 0; q < b->P; ++q) {
        edges += b->blk[q].nnz;
        sources += b->blk[q].n_src;
    }
    if (!even_rows(b->n_dst, edges, b->f_longest)) return Slices::kNo;
    const bool f32 = dtype == SAR_F32;
    const int lanes = slice_lanes(D);
    const int64_t slice = sources * D * (f32 ? 4 : 2), whole = slice * H;
    if (slice <= 3 << 20)
        return f32 && whole >= 12 << 20 && b->n_dst * H / (kWave / lanes) >= 10000 ? Slices::kFree : Slices::kNo;
    const int64_t least = scores_given ? (f32 ? 24 : 16) : f32 ? 20 : H > 1 ? 96 : 0;
    if (whole < least << 20) return Slices::kNo;
    return sweeps_pay(H, lanes, b->n_dst, edges, sources, scores_given && H >= slices::kXcds ? 5.0 : 2.0) ? Slices::kSwept
                                                                                                     : Slices::kNo;
}

// Backward: fp32 heads of 32, 64 or 128 values, in one or two slices of 128 values (the additions to ds), where sweeps pay
// and G is 28 MiB and more: on 3500 such graphs 0.87, 0.95, 1.07 of the time by rows (50 thousand destinations of 200
// thousand nodes, 8 x 32, 500 edges a row 3780 -> 3170 us); 16 to 24 MiB 1.02, 1.2, 1.5, less than 8 MiB 1.35 to 1.8.  bf16 4
// x 64 2000 / 2630.
bool bwd_by_slices(const sar_blocks_t* b, int dtype, int H, int D, int64_t edges)
{
    if (dtype != SAR_F32 || !(D == 32 || D == 64 || D == 128) || !(H * D == 128 || H * D == 256)) return false;
    if (b->n_dst * H * D * (int64_t)sizeof(float) < 28 << 20) return false;
    return even_rows(b->n_ft_wide, edges, b->ft_longest) &&
           sweeps_pay(H * D / 128, 32, b->n_ft_wide, edges, b->n_dst, 2.0);
}

}  // namespace

extern "C" int sar_gat_fwd_all(const sar_blocks_t* b, const void* const* Zq, const float* s,
                               const float* const* tq, const float* a_l, int dtype, int H, int D, float slope,
                               int act, void* out, float* L, void* stream)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_TRY(check_shape(dtype, H, D));
    SAR_TRY(check_act(act));
    if (!b->f_indptr) return sar::fail(SAR_ERR_STATE, "handle was built without SAR_BUILD_FUSED");
    if (b->n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(Zq && s && out && L, "a tensor argument is null");
    SAR_CHECK_ARG(tq || a_l, "either tq or a_l must be given");
    SAR_CHECK_ARG(aligned16(out) && aligned16(a_l), "out and a_l must be 16-byte aligned");
    for (int q = 0; q < b->P; ++q) {
        SAR_CHECK_ARG((Zq[q] && (!tq || tq[q])) || b->blk[q].nnz == 0, "Zq[%d] or tq[%d] is null", q, q);
        SAR_CHECK_ARG(aligned16(Zq[q]), "Zq[%d] must be 16-byte aligned", q);
    }
    hipStream_t st = sar::as_stream(stream);
    const Slices sl = fwd_by_slices(b, dtype, H, D, tq != nullptr);
    if (sl != Slices::kNo) {
        f256::FwdP p{};
        f256::Tabs tabs{};
        for (int q = 0; q < b->P; ++q) {
            tabs.Z[q] = Zq[q];
            tabs.t[q] = tq ? tq[q] : nullptr;
        }
        p.indptr = b->f_indptr;
        p.indices = b->f_indices;
        p.rows = reinterpret_cast<const uint32_t*>(b->f_rows);
        p.n_rows = b->n_dst;
        p.s = s;
        p.a_l = tq ? nullptr : a_l;
        p.out = out;
        p.L = L;
        p.H = p.ldh = H;
        p.D = D;
        p.ld = H * D;
        p.tag_shift = b->tag_shift;
        p.slope = slope;
        p.act = act;
        return sar::fwd_slices(dtype, p, tabs, sl == Slices::kSwept, st);
    }
    const HeadGroups hg = head_groups(dtype, H, D, fwd_pass(tq != nullptr, true));
    for (int g = 0; g < hg.n; ++g) {
        const size_t h0 = (size_t)hg.first(g), f0 = h0 * D;
        PtrTab zt{}, tt{};
        for (int q = 0; q < b->P; ++q) {
            zt.p[q] = shift(Zq[q], f0 * hg.fb);
            tt.p[q] = (tq && tq[q]) ? tq[q] + h0 : nullptr;
        }
        FwdArgs a{};
        a.indptr = b->f_indptr;
        a.indices = b->f_indices;
        a.rows = reinterpret_cast<const uint32_t*>(b->f_rows);
        a.n_rows = b->n_dst;   // the list ends with the destinations that have no in-edge: out = 0, L = -inf
        a.n_long = b->n_f_shared;
        a.s = s + h0;
        a.a_l = tq ? nullptr : a_l + f0;
        a.out = shift(out, f0 * hg.fb);
        a.L = L + h0;
        a.H = hg.count(g);
        a.n_hub = shared_hubs(b, (size_t)a.H * D * hg.fb, tq != nullptr);
        a.D = D;
        a.F = a.H * D;
        a.ldz = H * D;
        a.ldh = H;
        a.tag_shift = b->tag_shift;
        a.slope = slope;
        a.act = act;
        SAR_TRY(launch_fwd<true>(dtype, a, zt, tt, b->P, st));
    }
    return SAR_OK;
}

extern "C" int sar_gat_workspace_bytes(int64_t n_dst, int64_t n_src_max, int H, int D, size_t* bytes)
{
    SAR_CHECK_ARG(bytes != nullptr, "bytes is null");
    SAR_CHECK_ARG(n_dst >= 0 && n_src_max >= 0 && H > 0 && D > 0, "sizes must be non-negative, H and D positive");
    const int copies = ds_copies_for(n_dst, H);
    *bytes = workspace_bytes(256) + (copies > 1 ? (size_t)copies * ds_copy_bytes(n_dst, H) : 0) + slices_bytes(n_dst, H);
    return SAR_OK;
}

extern "C" int sar_gat_bwd_begin(const void* G, const void* out, const float* s, const float* L, int act,
                                 void* Gact, int dtype, float* rec, float* ds, int64_t n_dst, int H, int D,
                                 void* stream)
{
    SAR_TRY(check_shape(dtype, H, D));
    SAR_TRY(check_act(act));
    SAR_CHECK_ARG(n_dst >= 0, "n_dst is negative");
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(G && out && s && L && rec && ds, "a tensor argument is null");
    SAR_CHECK_ARG(aligned16(G) && aligned16(out) && aligned16(rec), "G, out and rec must be 16-byte aligned");
    SAR_CHECK_ARG(act == SAR_ACT_NONE || (Gact && aligned16(Gact)), "a non-linearity needs Gact (16-byte aligned)");
    const NodeGeo geo = node_geo(dtype, H, D);
    hipStream_t st = sar::as_stream(stream);
    for (int g = 0; g < geo.hg.n; ++g) {
        const size_t h0 = (size_t)geo.hg.first(g), f0 = h0 * D;
        const void* Gg = shift(G, f0 * geo.hg.fb);
        const void* og = shift(out, f0 * geo.hg.fb);
        float4* recg = reinterpret_cast<float4*>(rec) + h0;
        const unsigned grid = nodewise_grid(n_dst, geo.slots(g), begin_grid_most(n_dst, geo, g, D));
        SAR_DISPATCH_NODE(dtype, geo, (k_bwd_begin<T, kV, kL, kR><<<grid, kGatherThreads, 0, st>>>(
                                          static_cast<const T*>(Gg), static_cast<const T*>(og), s + h0, L + h0, recg,
                                          ds + h0, n_dst, geo.hg.count(g), D, H * D, H, act,
                                          static_cast<T*>(shift(Gact, f0 * geo.hg.fb)))));
        SAR_LAUNCH_CHECK();
    }
    return SAR_OK;
}

namespace {

int bwd_common_checks(const sar_blocks_t* b, int dtype, int H, int D, const void* G, const float* rec,
                      const float* a_l, const float* ds, const float* da_l, const void* work, size_t work_bytes)
{
    SAR_CHECK_ARG(b != nullptr, "handle is null");
    SAR_TRY(check_shape(dtype, H, D));
    if (!(b->flags & SAR_BUILD_TRANSPOSE))
        return sar::fail(SAR_ERR_STATE, "handle was built without SAR_BUILD_TRANSPOSE");
    // with no destination at all the destination-side tensors have no element (and may be null):
    // the sources still get their zero rows
    SAR_CHECK_ARG(a_l && da_l && (b->n_dst == 0 || (G && rec && ds)), "a tensor argument is null");
    SAR_CHECK_ARG(aligned16(G) && aligned16(rec) && aligned16(a_l), "G, rec and a_l must be 16-byte aligned");
    SAR_CHECK_ARG(work != nullptr && aligned16(work), "work is null or not 16-byte aligned");
    const size_t need = workspace_bytes(256);
    SAR_CHECK_ARG(work_bytes >= need, "work_bytes=%zu is below the %zu bytes required", work_bytes, need);
    return SAR_OK;
}

// Fields that do not depend on the block(s) or on the head group.
void fill_bwd_group(BwdScalars& a, const HeadGroups& hg, int g, int H, int D, const void* G, const float* rec,
                    const float* a_l, const DsTarget& ds, void* work, float slope)
{
    const size_t h0 = (size_t)hg.first(g), f0 = h0 * D;
    a.G = shift(G, f0 * hg.fb);
    a.rec = reinterpret_cast<const float4*>(rec) + h0;
    a.a_l = a_l + f0;
    a.ds = ds.base + h0;
    a.ds_stride = ds.stride;
    a.ds_copies = ds.copies;
    a.partial = static_cast<float*>(work);
    a.H = hg.count(g);
    a.D = D;
    a.F = a.H * D;
    a.ldz = H * D;
    a.ldh = H;
    a.slope = slope;
}

}  // namespace

extern "C" int sar_gat_bwd_block(const sar_blocks_t* b, int q, const void* Zq, const void* G, const float* tq,
                                 const float* rec, const float* a_l, int dtype, int H, int D, float slope,
                                 void* dZq, float* dtq, float* ds, float* da_l, void* work, size_t work_bytes,
                                 void* stream)
{
    SAR_TRY(bwd_common_checks(b, dtype, H, D, G, rec, a_l, ds, da_l, work, work_bytes));
    SAR_CHECK_ARG(q >= 0 && q < b->P, "block %d out of range [0,%d)", q, b->P);
    const sar::Block& k = b->blk[q];
    if (k.n_src == 0 || (sar::skips_untouched(b->flags) && k.n_t_rows == 0)) return SAR_OK;
    SAR_CHECK_ARG(Zq && dZq, "a tensor argument is null");
    SAR_CHECK_ARG(aligned16(Zq) && aligned16(dZq), "Zq and dZq must be 16-byte aligned");
    hipStream_t st = sar::as_stream(stream);
    DsTarget dst;
    const HeadGroups hg = head_groups(dtype, H, D, Pass::kBwd);
    SAR_TRY(ds_begin(dst, b->n_dst, ds_contended(k.hub, k.nnz, b->n_dst, H, D, hg.fb), H, ds, work, work_bytes, st));
    for (int g = 0; g < hg.n; ++g) {
        const size_t h0 = (size_t)hg.first(g), f0 = h0 * D;
        BwdArgs tabs{};
        tabs.t_indptr[0] = k.t_indptr;
        tabs.t_indices[0] = k.t_indices;
        tabs.Z[0] = shift(Zq, f0 * hg.fb);
        tabs.t[0] = tq ? tq + h0 : nullptr;
        tabs.dZ[0] = shift(dZq, f0 * hg.fb);
        tabs.dt[0] = dtq ? dtq + h0 : nullptr;
        tabs.rank[0] = (b->flags & SAR_BUILD_COMPACT) ? k.t_rank : nullptr;
        BwdScalars a{};
        a.rows = reinterpret_cast<const uint32_t*>(k.t_rows);
        // sources without edges come last and get dZ = 0, dt = 0, unless the handle skips them
        a.n_rows = sar::skips_untouched(b->flags) ? k.n_t_rows : k.n_src;
        a.n_long = k.n_t_shared;
        a.n_wide = k.n_t_wide;
        a.n_touched = k.n_t_rows;
        a.n_src_host = &k.n_src;
        a.n_blocks = 1;
        fill_bwd_group(a, hg, g, H, D, G, rec, a_l, dst, work, slope);
        SAR_TRY(launch_bwd<false>(dtype, tabs, a, da_l + f0, st));
    }
    return ds_end(dst, ds, st);
}

extern "C" int sar_gat_bwd_all(const sar_blocks_t* b, const void* const* Zq, const void* G,
                               const float* const* tq, const float* rec, const float* a_l, int dtype, int H,
                               int D, float slope, void* const* dZq, float* const* dtq, float* ds, float* da_l,
                               void* work, size_t work_bytes, void* stream)
{
    SAR_TRY(bwd_common_checks(b, dtype, H, D, G, rec, a_l, ds, da_l, work, work_bytes));
    SAR_CHECK_ARG(Zq && dZq, "a pointer table is null");
    if (b->P > SAR_MAX_BLOCKS)
        return sar::fail(SAR_ERR_UNSUPPORTED, "an all-blocks call takes at most %d blocks, the handle has %d: use the "
                         "per-block calls", SAR_MAX_BLOCKS, b->P);
    hipStream_t st = sar::as_stream(stream);
    for (int q = 0; q < b->P; ++q) {
        if (b->blk[q].n_src == 0 || (sar::skips_untouched(b->flags) && b->blk[q].n_t_rows == 0)) continue;
        SAR_CHECK_ARG(Zq[q] && (!tq || tq[q]) && dZq[q] && (!dtq || dtq[q]), "a tensor of block %d is null", q);
        SAR_CHECK_ARG(aligned16(Zq[q]) && aligned16(dZq[q]), "Zq[%d] and dZq[%d] must be 16-byte aligned", q, q);
    }
    const HeadGroups hg = head_groups(dtype, H, D, Pass::kBwd);
    DsTarget dst;
    int64_t nnz = 0, hub = 0;     // a frequent destination is frequent in every block
    for (int q = 0; q < b->P; ++q) {
        nnz += b->blk[q].nnz;
        hub += b->blk[q].hub;
    }
    SAR_TRY(ds_begin(dst, b->n_dst, ds_contended(hub, nnz, b->n_dst, H, D, hg.fb), H, ds, work, work_bytes, st));
    int64_t n_src_all[SAR_MAX_BLOCKS];
    for (int q = 0; q < b->P; ++q) n_src_all[q] = b->blk[q].n_src;

    // the sources of 8 edges and more by head slices, where that serves them better
    const int copies = ds_copies_for(b->n_dst, H);
    const size_t slices_at = workspace_bytes(256) + (copies > 1 ? (size_t)copies * ds_copy_bytes(b->n_dst, H) : 0);
    const size_t slices_need = slices_bytes(b->n_dst, H);
    const bool by_slices = slices_need > 0 && work_bytes >= slices_at + slices_need && bwd_by_slices(b, dtype, H, D, nnz);
    if (by_slices) {
        f256::BwdTabs tabs{};
        for (int q = 0; q < b->P; ++q) {
            const sar::Block& k = b->blk[q];
            if (k.n_src == 0) continue;
            tabs.t_indptr[q] = k.t_indptr;
            tabs.t_indices[q] = k.t_indices;
            tabs.Z[q] = Zq[q];
            tabs.t[q] = tq ? tq[q] : nullptr;
            tabs.dZ[q] = dZq[q];
            tabs.dt[q] = dtq ? dtq[q] : nullptr;
            tabs.rank[q] = (b->flags & SAR_BUILD_COMPACT) ? k.t_rank : nullptr;
        }
        f256::BwdP p{};
        p.rows = b->ft_rows;
        p.n_rows = b->n_ft_wide;
        p.G = G;
        p.rec = reinterpret_cast<const float4*>(rec);
        p.a_l = a_l;
        p.partial = static_cast<float*>(work);
        p.H = p.ldh = H;
        p.D = D;
        p.ld = H * D;
        p.tag_shift = b->tag_shift;
        p.slope = slope;
        SAR_TRY(sar::bwd_slices(p, tabs, b->n_dst, static_cast<char*>(work) + slices_at, ds, da_l, st));
    }
    for (int g = 0; g < hg.n; ++g) {
        const size_t h0 = (size_t)hg.first(g), f0 = h0 * D;
        BwdArgs tabs{};
        for (int q = 0; q < b->P; ++q) {
            const sar::Block& k = b->blk[q];
            if (k.n_src == 0) continue;
            tabs.t_indptr[q] = k.t_indptr;
            tabs.t_indices[q] = k.t_indices;
            tabs.Z[q] = shift(Zq[q], f0 * hg.fb);
            tabs.t[q] = tq ? tq[q] + h0 : nullptr;
            tabs.dZ[q] = shift(dZq[q], f0 * hg.fb);
            tabs.dt[q] = dtq ? dtq[q] + h0 : nullptr;
            tabs.rank[q] = (b->flags & SAR_BUILD_COMPACT) ? k.t_rank : nullptr;
        }
        BwdScalars a{};
        a.rows = b->ft_rows;
        a.n_rows = 0;
        for (int q = 0; q < b->P; ++q) a.n_rows += b->blk[q].n_src;
        if (sar::skips_untouched(b->flags)) a.n_rows = b->n_ft_rows;
        a.n_wide = b->n_ft_wide;
        a.n_touched = b->n_ft_rows;
        a.n_single = b->n_single;
        a.s_dst = b->s_dst;
        a.s_src = b->s_src;
        a.s_row = b->s_row;
        a.n_src_host = n_src_all;
        a.n_blocks = b->P;
        a.n_long = b->n_ft_shared;
        a.tag_shift = b->tag_shift;
        fill_bwd_group(a, hg, g, H, D, G, rec, a_l, dst, work, slope);
        a.wide_done = by_slices;
        SAR_TRY(launch_bwd<true>(dtype, tabs, a, da_l + f0, st));
    }
    return ds_end(dst, ds, st);
}

namespace {

// Scratch of the entry point that allocates nothing: one row of partial sums of da_r per
// workgroup of k_bwd_end (at most kMaxPersistentWGs workgroups, at most 512 values per launch).
// Host code never uses the array's name as an address: the device address is looked up once
// per device (scratch_of) and passed to the kernels like any caller workspace.
constexpr size_t kScratchFloats = (size_t)kMaxPersistentWGs * 512;
static __device__ __align__(256) float scratch[kScratchFloats];

constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (each device holds its own copy).
int scratch_of(float** out)
{
    int dev = -1;
    SAR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return sar::fail(SAR_ERR_UNSUPPORTED, "device ordinal %d is beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        SAR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return sar::fail(SAR_ERR_HIP, "hipGetSymbolAddress returned a null address for the scratch array");
        g_scratch_ptr[dev] = static_cast<float*>(p);
    }
    *out = g_scratch_ptr[dev];
    return SAR_OK;
}

// partial: room for one row of sums (the launch's heads) per workgroup; partial_floats = its size in values.
int bwd_end_impl(const void* Zdst, const float* ds, const float* a_r, const void* dZadd,
                 const int32_t* dZadd_rank, void* dZdst, float* da_r, int dtype, int64_t n_dst, int H, int D, float* partial, size_t partial_floats,
                 hipStream_t st)
{
    const NodeGeo geo = node_geo(dtype, H, D);
    for (int g = 0; g < geo.hg.n; ++g) {
        const int Hg = geo.hg.count(g), Fg = Hg * D;
        const size_t h0 = (size_t)geo.hg.first(g), f0 = h0 * D;
        const unsigned grid = nodewise_grid(n_dst, geo.slots(g));
        if ((size_t)grid * Fg > partial_floats)
            return sar::fail(SAR_ERR_UNSUPPORTED, "%u workgroups x %d partial sums exceed the %zu values of scratch",
                             grid, Fg, partial_floats);
        SAR_DISPATCH_NODE(dtype, geo, (k_bwd_end<T, kV, kL, kR><<<grid, kGatherThreads, 0, st>>>(
                                          static_cast<const T*>(Zdst) + f0, ds + h0, a_r + f0,
                                          dZadd ? static_cast<const T*>(dZadd) + f0 : nullptr, dZadd_rank,
                                          dZdst ? static_cast<T*>(dZdst) + f0 : nullptr, partial, n_dst, Hg, D, H * D, H)));
        SAR_LAUNCH_CHECK();
        SAR_TRY(reduce_partials(partial, (int)grid, Fg, da_r + f0, st));
    }
    return SAR_OK;
}

int bwd_end_checks(const void* Zdst, const float* ds, const float* a_r, const void* dZadd,
                   const int32_t* dZadd_rank, void* dZdst, float* da_r, int dtype, int64_t n_dst, int H, int D)
{
    SAR_CHECK_ARG(!dZadd_rank || (dZadd && dZadd != dZdst), "dZadd_rank needs a dZadd that is not dZdst");
    SAR_TRY(check_shape(dtype, H, D));
    SAR_CHECK_ARG(n_dst >= 0, "n_dst is negative");
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(Zdst && ds && a_r && da_r, "a tensor argument is null");
    SAR_CHECK_ARG(aligned16(Zdst) && aligned16(dZdst) && aligned16(dZadd),
                  "Zdst, dZadd and dZdst must be 16-byte aligned");
    return SAR_OK;
}

}  // namespace

extern "C" int sar_gat_bwd_end(const void* Zdst, const float* ds, const float* a_r, const void* dZadd,
                               const int32_t* dZadd_rank, void* dZdst, float* da_r, int dtype, int64_t n_dst,
                               int H, int D, void* work, size_t work_bytes, void* stream)
{
    SAR_TRY(bwd_end_checks(Zdst, ds, a_r, dZadd, dZadd_rank, dZdst, da_r, dtype, n_dst, H, D));
    if (n_dst == 0) return SAR_OK;
    SAR_CHECK_ARG(work != nullptr && aligned16(work), "work is null or not 16-byte aligned");
    const size_t need = workspace_bytes(256);
    SAR_CHECK_ARG(work_bytes >= need, "work_bytes=%zu is below the %zu bytes required", work_bytes, need);
    return bwd_end_impl(Zdst, ds, a_r, dZadd, dZadd_rank, dZdst, da_r, dtype, n_dst, H, D,
                        static_cast<float*>(work), work_bytes / sizeof(float), sar::as_stream(stream));
}

extern "C" int sar_gat_bwd_end_noalloc(const void* Zdst, const float* ds, const float* a_r, const void* dZadd,
                                       const int32_t* dZadd_rank, void* dZdst, float* da_r, int dtype,
                                       int64_t n_dst, int H, int D, void* stream)
{
    SAR_TRY(bwd_end_checks(Zdst, ds, a_r, dZadd, dZadd_rank, dZdst, da_r, dtype, n_dst, H, D));
    if (n_dst == 0) return SAR_OK;
    float* partial = nullptr;
    SAR_TRY(scratch_of(&partial));
    return bwd_end_impl(Zdst, ds, a_r, dZadd, dZadd_rank, dZdst, da_r, dtype, n_dst, H, D, partial,
                        kScratchFloats, sar::as_stream(stream));
}
