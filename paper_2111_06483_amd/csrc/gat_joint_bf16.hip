// Small backward calls of bf16 rows.
#include "gat_joint_launch.h"

int sar::bwd_joint_bf16(const f256::BwdTabs& t, const f256::BwdP& p, const joint::Work& w, int* grid, hipStream_t st)
{
    return w.all ? by_lanes<bf16_t, true>(t, p, w, grid, st) : by_lanes<bf16_t, false>(t, p, w, grid, st);
}
