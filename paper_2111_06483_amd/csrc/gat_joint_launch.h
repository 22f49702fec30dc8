// The small backward calls' launch (gat_joint.h), included once for each type of the rows: each is a file of its own, because
// together they take the compiler two minutes.
#pragma once

#include "gat_joint.h"

#include "sar_internal.h"

namespace sar {

namespace {

using joint::Grid;
using joint::Lanes;
using joint::Work;

template <typename T, int LPH, bool ALL, Lanes L>
int launch(const f256::BwdTabs& t, const f256::BwdP& p, Work w, int* grid, hipStream_t st)
{
    constexpr bool SLOTS = L == Lanes::kSlots;
    auto kernel = joint::k_gat_bwd_joint<T, LPH, ALL, L>;
    static const int resident = resident_workgroups(kernel);
    const int64_t per_wg = (int64_t)(SLOTS ? w.n_slots : (LPH >= 8 ? 8 : 4) / 2) * kWavesPerWG;
    Grid g{};
    // (a part that would go round asks for more workgroups than there are)
    if (p.n_rows > 0) g.wide = (int)persistent_grid_for(p.n_rows, p.n_long, resident + 1);
    for (int k = 0; k < 2; ++k) {
        const int64_t n = w.piece[k][1] - w.piece[k][0];
        if (n > 0) g.few[k] = (int)grid_of(n, per_wg, resident + 1);
    }
    if (w.single.n > 0) {
        unsigned n = 0;
        const int64_t once = (int64_t)(resident / 2) * kWavesPerWG * kWave;
        w.single = single_list(w.single, resident / 2, n);
        g.single = w.single.n > once ? resident + 1 : (int)n;
    }
    *grid = 0;
    const int total = g.total(), parts = (g.wide > 0) + (g.few[0] > 0) + (g.few[1] > 0) + (g.single > 0);
    if (parts < 2 || total > resident) return SAR_OK;
    kernel<<<(unsigned)total, kGatherThreads, 0, st>>>(t, p, w, g);
    SAR_LAUNCH_CHECK();
    *grid = total;
    return SAR_OK;
}

template <typename T, bool ALL>
int by_lanes(const f256::BwdTabs& t, const f256::BwdP& p, const Work& w, int* grid, hipStream_t st)
{
#define SAR_JOINT(LPH, L) \
    case LPH: return launch<T, LPH, ALL, Lanes::L>(t, p, w, grid, st)
    switch (w.lanes) {
        case Lanes::kExact:
            switch (w.lph) { SAR_JOINT(4, kExact); SAR_JOINT(8, kExact); SAR_JOINT(16, kExact); SAR_JOINT(32, kExact); SAR_JOINT(64, kExact); }
            break;
        case Lanes::kPadded:
            switch (w.lph) { SAR_JOINT(8, kPadded); SAR_JOINT(16, kPadded); SAR_JOINT(32, kPadded); SAR_JOINT(64, kPadded); }
            break;
        case Lanes::kSlots:
            if constexpr (ALL) {
                switch (w.lph) { SAR_JOINT(4, kSlots); SAR_JOINT(8, kSlots); SAR_JOINT(16, kSlots); SAR_JOINT(32, kSlots); }
            }
            break;
    }
#undef SAR_JOINT
    return fail(SAR_ERR_STATE, "no joint backward kernel for %d lanes a head", w.lph);
}

}  // namespace

}  // namespace sar
