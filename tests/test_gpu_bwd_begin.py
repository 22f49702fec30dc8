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
