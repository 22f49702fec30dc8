"""The backward pass's node-wise beginning on both sides of the size from which every wavefront takes its rows once: records and
cleared ds against 64 bits, with and without ReLU (in place too)."""
import math

import pytest
import torch

from paper_2111_06483_amd import sar

pytestmark = pytest.mark.gpu


# two arrays of 256 MiB in all are 131072 rows of 256 fp32 values; whole heads, ragged ones, several launches of heads
@pytest.mark.parametrize("n,H,D,dtype", [(131_072, 4, 64, torch.float32), (131_073, 4, 64, torch.float32),
                                         (300_007, 8, 32, torch.bfloat16), (90_001, 4, 100, torch.float32),
                                         (720_001, 1, 47, torch.float32), (720_001, 3, 12, torch.float32)])
@pytest.mark.parametrize("act", [sar.SAR_ACT_NONE, sar.SAR_ACT_RELU])
def test_records(n, H, D, dtype, act):
    g = torch.Generator(device="cuda").manual_seed(n + D)
    randn = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    G, out, s, L = randn(n, H, D).to(dtype), randn(n, H, D).to(dtype), randn(n, H), randn(n, H)
    if act == sar.SAR_ACT_RELU:
        out = out.clamp_(min=0)
    rec, ds = torch.full((n, H, 4), 7.0, device="cuda"), torch.full((n, H), 7.0, device="cuda")
    masked = G * (out > 0) if act == sar.SAR_ACT_RELU else G
    products = masked.double() * out.double()
    want, room = products.sum(2), products.abs().sum(2) * D * 2.0 ** -23
    Gact = G if act == sar.SAR_ACT_RELU else None
    sar.sar_gat_bwd_begin(G, out, s, L, rec, ds, act, Gact)
    if act == sar.SAR_ACT_RELU:
        assert torch.equal(G, masked)
    assert not ds.any() and not rec[..., 3].any()
    assert ((rec[..., 2].double() - want).abs() <= room).all()
    for k, t in ((0, s), (1, L)):
        assert ((rec[..., k].double() - t.double() / math.log(2.0)).abs() <= t.double().abs() * 2.0 ** -21).all()


# arrays beyond the memory-side cache: wavefronts that move little at a time and rows of unaligned pieces stay with a resident grid,
# as arrays do that a part of fits it; records count, and launch by launch where heads are shared among several
@pytest.mark.parametrize("mib,H,D,dtype,once", [
    (400, 2, 100, torch.bfloat16, False), (1200, 2, 100, torch.bfloat16, False), (400, 1, 47, torch.bfloat16, False),
    (1200, 1, 47, torch.float32, False), (400, 5, 40, torch.bfloat16, False), (400, 4, 20, torch.float32, False),
    (280, 4, 64, torch.float32, False), (280, 8, 32, torch.bfloat16, True), (200, 8, 8, torch.float32, False),
    (240, 8, 8, torch.float32, True), (400, 4, 64, torch.float32, True), (400, 8, 32, torch.bfloat16, True),
    (400, 3, 12, torch.float32, True), (400, 2, 100, torch.float32, True), (400, 8, 4, torch.bfloat16, True),
    (500, 4, 100, torch.float32, False), (1000, 4, 100, torch.float32, True)])
def test_which_rows_are_taken_once(mib, H, D, dtype, once):
    from tests import gpu_util as gu
    n = (mib << 20) // (2 * H * D * (4 if dtype == torch.float32 else 2))
    G, out, s, L = (torch.ones(n, *shape, device="cuda") for shape in ((H, D), (H, D), (H,), (H,)))
    G, out = G.to(dtype), out.to(dtype)
    rec, ds = torch.empty(n, H, 4, device="cuda"), torch.empty(n, H, device="cuda")
    grids = [wgs for name, wgs in gu.launches_of(lambda: sar.sar_gat_bwd_begin(G, out, s, L, rec, ds)) if "k_bwd_begin" in name]
    assert grids and all((g > 2048) == once for g in grids), grids


# beyond the size: the last wavefront full, with one row, and with some of its slots
@pytest.mark.parametrize("n,H,D,dtype", [(163_841, 4, 64, torch.float32), (330_003, 8, 32, torch.bfloat16),
                                         (1_200_001, 3, 12, torch.float32), (220_001, 4, 100, torch.float32),
                                         (2_700_000, 8, 4, torch.bfloat16)])
@pytest.mark.parametrize("act", [sar.SAR_ACT_NONE, sar.SAR_ACT_RELU])
def test_records_of_rows_taken_once(n, H, D, dtype, act):
    test_records(n, H, D, dtype, act)
