"""Rows far longer than a workgroup's share of the edges, in the forward pass over all blocks: those of 1024 edges and more are
shared by twelve wavefronts.  Lengths around that line, around whole and ragged teams of it and below it, against sums
in fp64."""
import pytest
import torch

from paper_2111_06483_amd import sar

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 9000, 1024, 1023, 5, 1500, 4097, 128, 127, 700, 768, 1025, 64, 300, 0, 200, 150, 2, 1536, 511, 513]
N, P = 12_000, 3
# a row's terms pass through at most 9000 / 4 additions one after another, each off by 2^-24 of what is summed: eight
# standard deviations of that walk (an edge left out of the longest row is 1e-4)
TOL = 8 * (9000 / 4) ** 0.5 * 2.0 ** -24


def graph(seed, only_few):
    g = torch.Generator().manual_seed(seed)
    lengths = [5, 0, 5000, 1] if only_few else LENGTHS + [3] * 40
    dst = torch.cat([torch.full((n,), i, dtype=torch.int64) for i, n in enumerate(lengths)])
    src = torch.cat([torch.randperm(N, generator=g)[:n] for n in lengths])
    own = len(lengths)
    part = torch.cat([torch.zeros(own, dtype=torch.int32), 1 + (torch.arange(N - own) * 2 // (N - own)).to(torch.int32)])
    b = sar.sar_blocks_build(src.cuda(), dst.cuda(), part.cuda(), P, 0, sar.SAR_BUILD_FUSED | sar.SAR_BUILD_TRANSPOSE)
    return b, src.cuda(), dst.cuda(), own, g


def check(got, want, tol):
    assert torch.isfinite(got).all()
    assert float((got.double() - want).abs().max()) <= tol * float(want.abs().max())


@pytest.mark.parametrize("rows,length,filler,few,many", [(400, 2100, 0, 12, 12), (400, 2100, 300_000, 4, 12),
                                                         (60, 2100, 0, 4, 4), (2, 4200, 0, 12, 12), (400, 1100, 0, 4, 4)])
def test_which_workgroups_share_rows(rows, length, filler, few, many):
    """Rows far longer than a workgroup's share of all edges and of one to two shares (there rows of 1 KiB stay with workgroups
    of four wavefronts); too few of 2048 edges, two of 4096, and none as long as that."""
    counts = torch.cat([torch.full((rows,), length), torch.full((filler,), 6)]).cuda()
    n, g = counts.numel(), torch.Generator(device="cuda").manual_seed(1)
    n += 5000               # (sources enough)
    dst = torch.repeat_interleave(torch.arange(n - 5000, device="cuda"), counts)
    src = torch.randint(0, n, (dst.numel(),), generator=g, device="cuda")
    b = sar.sar_blocks_build(src, dst, torch.zeros(n, dtype=torch.int32, device="cuda"), 1, 0, sar.SAR_BUILD_FUSED)
    for dtype, H, D, waves in ((torch.float32, 4, 64, few), (torch.bfloat16, 4, 64, many), (torch.float32, 2, 100, many)):
        Z, a_l = torch.randn(n, H, D, generator=g, device="cuda").to(dtype), torch.randn(H, D, generator=g, device="cuda")
        s, out, L = torch.randn(n, H, generator=g, device="cuda"), torch.empty_like(Z), torch.empty(n, H, device="cuda")
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
            sar.sar_gat_fwd_all(b, [Z], s, None, a_l, 0.2, out, L, sar.SAR_ACT_NONE)
            torch.cuda.synchronize()
        assert any("k_gat_fwd_f256" in e.name and ", %d>" % waves in e.name for e in p.events())


@pytest.mark.parametrize("only_few", [False, True])
@pytest.mark.parametrize("H,D", [(4, 64), (8, 32), (1, 256), (16, 16), (2, 96), (6, 40), (2, 100)])
@pytest.mark.parametrize("dtype,shipped,relu", [(torch.float32, False, False), (torch.float32, True, True),
                                                (torch.bfloat16, False, True), (torch.bfloat16, True, False)])
def test_attention(H, D, dtype, shipped, relu, only_few):
    b, src, dst, own, g = graph(H * D, only_few)
    Z = torch.randn(N, H, D, generator=g).to(dtype).cuda()
    a_l, a_r = (torch.randn(H, D, generator=g).cuda() / D ** 0.5 for _ in range(2))
    starts = [0, own, own + (N - own + 1) // 2, N]
    assert [b.n_src(q) for q in range(P)] == [starts[q + 1] - starts[q] for q in range(P)]
    Zs = [Z[starts[q]:starts[q + 1]].clone() for q in range(P)]
    s = torch.empty(own, H, device="cuda")
    sar.sar_gat_scores(Zs[0], a_r, s)
    tq = [torch.empty(len(z), H, device="cuda") for z in Zs]
    for z, t in zip(Zs, tq):
        sar.sar_gat_scores(z, a_l, t)
    out, L = torch.full((own, H, D), 7.0, device="cuda", dtype=dtype), torch.full((own, H), 7.0, device="cuda")
    sar.sar_gat_fwd_all(b, Zs, s, tq if shipped else None, a_l, 0.2, out, L, sar.SAR_ACT_RELU if relu else sar.SAR_ACT_NONE)
    e = torch.nn.functional.leaky_relu(s.double()[dst] + torch.cat(tq).double()[src], 0.2)
    total = torch.zeros(own, H, dtype=torch.float64, device="cuda").index_add_(0, dst, e.exp())
    want = torch.zeros(own, H, D, dtype=torch.float64, device="cuda")
    want.index_add_(0, dst, e.exp()[:, :, None] * Z.double()[src])
    want = torch.where(total[:, :, None] > 0, want / total[:, :, None], 0.0)
    check(out, want.clamp(min=0) if relu else want, TOL if dtype == torch.float32 else 2.0 ** -8)
    some = total > 0
    check(L[some], total.log()[some], TOL)
    assert L[~some].isneginf().all()
