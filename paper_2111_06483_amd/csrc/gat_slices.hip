// Launches of the kernels for dense graphs (gat_slices.h).
#include "gat_slices.h"

#include <algorithm>

namespace {

using namespace sar;

// Workgroups that serve `rows` rows: a multiple of the XCDs.  With barriers there are as many as four times the CUs, so
// that a CU takes another when its own ends (one runs at a time, by registers); without, as many as run at once.
constexpr int kMostSynced = 1024;
template <bool SYNC>
unsigned grid_of(int resident, int64_t rows, int sets, int slots)
{
    const int parts = sets < slices::kXcds ? slices::kXcds / sets : 1;                 // XCDs that share a set's rows
    const int64_t per_wg = (int64_t)slices::kWaves<SYNC> * slots * parts;
    const int64_t want = (rows + per_wg - 1) / per_wg;
    const int64_t enough = (SYNC ? kMostSynced : resident) / slices::kXcds;
    return (unsigned)(std::max<int64_t>(1, std::min<int64_t>(want, enough)) * slices::kXcds);
}

template <typename T, int LPH, bool FLY, bool PAD, bool SYNC>
int launch_fwd(const f256::FwdP& p, const f256::Tabs& tabs, hipStream_t st)
{
    auto fn = slices::k_gat_fwd_slices<T, LPH, FLY, PAD, SYNC>;
    static const int resident = SYNC ? 0 : resident_workgroups(fn);
    const unsigned grid = grid_of<SYNC>(resident, p.n_rows, p.H, kWave / LPH);
    fn<<<grid, slices::kThreads<SYNC>, 0, st>>>(p, tabs);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <int LPH, int HS>
int launch_bwd(const f256::BwdP& p, const f256::BwdTabs& tabs, int64_t n_dst, void* scratch, float* ds, float* da_l,
               hipStream_t st)
{
    auto fn = slices::k_gat_bwd_slices<LPH, HS>;
    const int64_t total = n_dst * p.H;
    const unsigned g_all = (unsigned)std::min<int64_t>((total + 255) / 256, kMaxPersistentWGs);
    float4* rec = static_cast<float4*>(scratch);
    float* ds_sets = reinterpret_cast<float*>(rec + total);
    slices::k_slices_begin<HS><<<g_all, 256, 0, st>>>(p.rec, rec, ds_sets, n_dst, p.H);
    SAR_LAUNCH_CHECK();
    const int sets = p.H / HS, width = HS * p.D;
    static_assert(kMostSynced <= kMaxPersistentWGs, "a row of partial sums for every workgroup in the caller's scratch");
    const unsigned grid = grid_of<true>(0, p.n_rows, sets, kWave / (LPH * HS));
    fn<<<grid, slices::kThreads<true>, 0, st>>>(tabs, p, slices::SetP{rec, ds_sets, n_dst});
    SAR_LAUNCH_CHECK();
    slices::k_slices_da<<<(unsigned)(p.H * p.D), 256, 0, st>>>(p.partial, (int)(grid / slices::kXcds), sets, width, da_l);
    SAR_LAUNCH_CHECK();
    slices::k_slices_end<HS><<<g_all, 256, 0, st>>>(ds_sets, ds, n_dst, p.H);
    SAR_LAUNCH_CHECK();
    return SAR_OK;
}

template <typename T, bool FLY, bool SYNC>
int fwd_typed(const f256::FwdP& p, const f256::Tabs& tabs, hipStream_t st)
{
    constexpr bool F32 = sizeof(T) == 4;
    if (F32 && p.D == 32) return launch_fwd<float, 8, FLY, false, SYNC>(p, tabs, st);
    if (p.D == 64) return launch_fwd<T, 16, FLY, false, SYNC>(p, tabs, st);
    if (F32 && p.D < 64) return launch_fwd<float, 16, FLY, true, SYNC>(p, tabs, st);
    if (p.D == 128) return launch_fwd<T, 32, FLY, false, SYNC>(p, tabs, st);
    return launch_fwd<T, 32, FLY, true, SYNC>(p, tabs, st);
}

}  // namespace

namespace sar {

int fwd_slices(int dtype, const f256::FwdP& p, const f256::Tabs& tabs, bool sync, hipStream_t st)
{
    auto with = [&](auto fly, auto synced) {
        constexpr bool FLY = decltype(fly)::value, SYNC = decltype(synced)::value;
        return dtype == SAR_F32 ? fwd_typed<float, FLY, SYNC>(p, tabs, st) : fwd_typed<bf16_t, FLY, SYNC>(p, tabs, st);
    };
    if (p.a_l) return sync ? with(std::true_type{}, std::true_type{}) : with(std::true_type{}, std::false_type{});
    return sync ? with(std::false_type{}, std::true_type{}) : with(std::false_type{}, std::false_type{});
}

int bwd_slices(const f256::BwdP& p, const f256::BwdTabs& tabs, int64_t n_dst, void* scratch, float* ds, float* da_l,
               hipStream_t st)
{
    if (p.D == 32) return launch_bwd<8, 4>(p, tabs, n_dst, scratch, ds, da_l, st);
    if (p.D == 64) return launch_bwd<16, 2>(p, tabs, n_dst, scratch, ds, da_l, st);
    return launch_bwd<32, 1>(p, tabs, n_dst, scratch, ds, da_l, st);
}

}  // namespace sar
