// The backward pass of a small call as one launch.
//
// Sources of 8 edges and more, the others, and those of one edge have kernels of their own, which do not depend on each other.
// In a small call none of them fills the chip, and each is a launch and a chain of loads of 5 to 10 us.  Here their workgroups
// are one launch where there are two parts at least and all workgroups that they ask for are resident at once; beyond that the kernels
// run one after the other, each with the registers it needs.  (Kernels one after the other / together, us: 8 x 32 over 12 thousand
// edges 27 / 14, 2 x 100 over 60 thousand 26 / 14, 5 x 40 of two launches over 100 thousand 64 / 19; a step of 2 x 100 over 15 thousand
// nodes in 9 blocks 74 / 63.)  Parts that go round lose by it, and so does a part alone: this kernel holds three or four workgroups
// a CU, the others up to seven, and gives single-edge sources half the chip.  (800 wide sources and 1600 of three edges beside single-edge ones,
// bf16 4 x 64: 65 thousand 36 / 31, 131 thousand 47 / 47, 262 thousand 81 / 94, 2 million 465 / 597; fp32 8 x 32 49 / 40, 80 / 83, 144 / 137,
// 878 / 906.  Sources of three edges alone, bf16 4 x 64: 30 thousand 26 / 28, 300 thousand 143 / 158, 2 million 859 / 976.)
#pragma once

#include "gat_slots.h"

namespace sar {

// Workgroups for `items` pieces of work.
inline unsigned grid_of(int64_t items, int64_t per_wg, int resident)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + per_wg - 1) / per_wg, resident));
}

// The list of single-edge sources: a wavefront takes 64 entries at a time, eight after the other by eight, where that many
// are there for each; of a short list it takes 32, 16 or 8, down to one round for every wavefront the chip holds (20 thousand
// entries, 64 at a time by 320 wavefronts: 20 us; 8 at a time by 2500: 6 us).
inline f256::SingleP single_list(f256::SingleP s, int resident, unsigned& grid)
{
    s.per = kWave;
    while (s.per > 8 && s.n < (int64_t)resident * kWavesPerWG * s.per) s.per /= 2;
    grid = grid_of(s.n, (int64_t)s.per * kWavesPerWG, resident);
    return s;
}

namespace joint {

enum class Lanes { kExact, kPadded, kSlots };      // (slots: with a list of single-edge sources)

// What a call has to do: wide sources (p.n_rows, p.n_long of the list), pieces [from, to) of the list for the others, the list of
// those of one edge.
struct Work {
    int64_t piece[2][2];
    f256::SingleP single;       // n = 0: none
    int n_slots;
    int lph;
    Lanes lanes;
    bool all;
};

// The launch's workgroups: the first `wide`, then few[0], few[1], the rest for single-edge sources.
struct Grid {
    int wide, few[2], single;
    int total() const { return wide + few[0] + few[1] + single; }
};

template <typename T, int LPH, bool ALL, Lanes L>
__global__ __launch_bounds__(kGatherThreads) void k_gat_bwd_joint(f256::BwdTabs tabs, f256::BwdP a, Work w, Grid g)
{
    constexpr bool SLOTS = L == Lanes::kSlots, PAD = L != Lanes::kExact;
    constexpr int B = LPH >= 8 ? 8 : 4;
    float* const row = a.partial + (int64_t)blockIdx.x * f256::kF;
    int b = (int)blockIdx.x;
    if (b < g.wide) {
        if constexpr (SLOTS)
            slots::bwd_wide<T, LPH, ALL, false>(tabs, a, w.n_slots, b, g.wide, row);
        else
            f256::bwd_wide<T, LPH, B, ALL, PAD>(tabs, a, b, g.wide, row);
    } else if ((b -= g.wide) < g.few[0] + g.few[1]) {
        const int k = b < g.few[0] ? 0 : 1;
        b -= k ? g.few[0] : 0;
        if constexpr (SLOTS)
            slots::bwd_few<T, LPH, ALL, false>(tabs, a, w.n_slots, w.piece[k][0], w.piece[k][1], b, g.few[k], row);
        else
            f256::bwd_few<T, LPH, ALL, PAD>(tabs, a, w.piece[k][0], w.piece[k][1], b, g.few[k], row);
    } else {
        if constexpr (ALL)
            f256::bwd_single<T, LPH, PAD>(tabs, a, w.single, b - g.few[0] - g.few[1], g.single, row);
    }
}

}  // namespace joint

// Takes a call if it is small enough: *grid workgroups have each left a row of 256 partial sums of da_l.  *grid = 0: not taken.
int bwd_joint(int dtype, const f256::BwdTabs& t, const f256::BwdP& p, const joint::Work& w, int* grid, hipStream_t st);
int bwd_joint_bf16(const f256::BwdTabs& t, const f256::BwdP& p, const joint::Work& w, int* grid, hipStream_t st);

}  // namespace sar
