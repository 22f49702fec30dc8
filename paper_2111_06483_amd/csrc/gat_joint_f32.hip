// Small backward calls of fp32 rows.
#include "gat_joint_launch.h"

int sar::bwd_joint(int dtype, const f256::BwdTabs& t, const f256::BwdP& p, const joint::Work& w, int* grid, hipStream_t st)
{
    if (dtype == SAR_BF16) return bwd_joint_bf16(t, p, w, grid, st);
    return w.all ? by_lanes<float, true>(t, p, w, grid, st) : by_lanes<float, false>(t, p, w, grid, st);
}
