"""How many workgroups take the sources of 8 edges and more: two a CU where they are many and their rows long fp32 rows, all that
are resident else."""
import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

TWO_PER_CU = 512


@pytest.mark.parametrize("n,H,D,dtype,two", [
    (140_000, 4, 64, torch.float32, True), (140_000, 3, 64, torch.float32, True), (140_000, 3, 56, torch.float32, True),
    (140_000, 4, 40, torch.float32, False), (140_000, 6, 36, torch.float32, False), (120_000, 4, 64, torch.float32, False),
    (140_000, 4, 64, torch.bfloat16, False)])
def test_workgroups(n, H, D, dtype, two):
    n_dst, deg = 3000, 8
    first = (torch.arange(n, device="cuda") * 31).repeat_interleave(deg)
    dst = (first + 7 * (torch.arange(n * deg, device="cuda") % deg)) % n_dst
    src = n_dst + torch.arange(n, device="cuda").repeat_interleave(deg)
    part = torch.cat([torch.zeros(n_dst), torch.ones(n)]).to(torch.int32).cuda()
    b = sar.sar_blocks_build(src, dst, part, 2, 0, 3 | sar.SAR_BUILD_COMPACT)
    Zs = [torch.randn(b.n_src(q), H, D, device="cuda").to(dtype) for q in range(2)]
    a_l = torch.randn(H, D, device="cuda")
    fw = gu.gat_fwd_all(b, Zs[0], Zs, a_l, a_l, 0.2)
    G = torch.randn(n_dst, H, D, device="cuda").to(dtype)
    rec, ds, da_l = torch.empty(n_dst, H, 4, device="cuda"), torch.empty(n_dst, H, device="cuda"), torch.zeros(H, D, device="cuda")
    sar.sar_gat_bwd_begin(G, fw.out, fw.s, fw.L, rec, ds)
    dZs = [torch.empty(b.n_err_rows(q), H, D, dtype=dtype, device="cuda") for q in range(2)]
    work = torch.empty(sar.sar_gat_workspace_bytes(n_dst, n, H, D) // 4, device="cuda")
    grids = [wgs for name, wgs in gu.launches_of(lambda: sar.sar_gat_bwd_all(b, Zs, G, None, rec, a_l, 0.2, dZs, None, ds, da_l, work))
             if "k_gat_bwd_f256" in name]
    assert grids and all((g == TWO_PER_CU) == two and g >= TWO_PER_CU for g in grids), grids
    b.close()
