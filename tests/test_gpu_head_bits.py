"""Last bits inside a head: lanes that hold one value of a head agree on it, the source score halves that the
kernels form in flight are those of sar_gat_scores, and a score of exactly zero is one in every kernel."""
import numpy as np
import pytest
import torch

from oracle import sar_oracle as orc
from paper_2111_06483_amd import sar
from tests import gpu_util as gu
from tests.helpers import rel_err, tiny_graph

pytestmark = pytest.mark.gpu
SLOPE = 0.2


def blocks_and_parameters(H, D, flags=0, drop=None):
    """Rows of 0 to some hundreds of edges; sources of one edge, of few and of many.  drop: leave out the edges of
    this source of block 0."""
    rng = np.random.default_rng(H * 1000 + D)
    src, dst, part = tiny_graph(rng, 1_500, 12_000, 2, simple=False)
    hub = rng.random(src.size) < 0.3
    src, dst = np.where(hub, src % 40, src), np.where(hub, dst, dst)
    more = np.flatnonzero(part == 0)[rng.integers(0, 3, 2_000)]
    src, dst = np.concatenate([src, rng.integers(0, 1_500, 2_000)]), np.concatenate([dst, more])
    if drop is not None:
        keep = src != np.flatnonzero(part == 0)[drop]
        src, dst = src[keep], dst[keep]
    b = gu.build_blocks(src, dst, part, 2, 0, flags=sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | flags)
    want_b, _ = orc.build_blocks(src, dst, part, 2, 0)
    bound = np.sqrt(6.0 / (D + 1))
    a_l, a_r = (torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda() for _ in range(2))
    return rng, b, want_b, a_l, a_r


# 16, 32 and 64 lanes of 4 values, whole and ragged heads; the last lane of a ragged head opens a quad (33, 49),
# an eight (65, 34) or stands inside one (47, 50)
@pytest.mark.parametrize("H,D", [(4, 64), (1, 256), (2, 100), (3, 33), (1, 34), (1, 47),
                                 (2, 50), (1, 126)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("batched", [False, True])
def test_lanes_of_a_head_agree(H, D, dtype, batched):
    """Rows and parameters that are constant along a head give results that are, bit for bit."""
    rng, b, _, a_l, a_r = blocks_and_parameters(H, D)
    a_l = a_l[:, :1].expand(H, D).contiguous()
    row = lambda n: torch.from_numpy(rng.standard_normal((n, H, 1)).astype(np.float32)).to(dtype).cuda().expand(n, H, D).contiguous()
    Zs, G = [row(b.n_src(q)) for q in range(2)], row(b.n_dst)
    fw = (gu.gat_fwd_all if batched else gu.gat_fwd_stream)(b, Zs[0], Zs, a_l, a_r, SLOPE, fly=True)
    g = gu.gat_bwd(b, Zs[0], Zs, G, a_l, a_r, SLOPE, fw, batched, fly=True)
    for name, t in [("out", fw.out)] + [("dZ%d" % q, z) for q, z in enumerate(g.dZs)]:
        assert torch.equal(t, t[:, :, :1].expand_as(t)), name
    b.close()


# fp32 heads of 4, 8, 16 ... values and, in both types, widths that are no multiple of 4
@pytest.mark.parametrize("dtype,H,D", [(torch.float32, 4, 64), (torch.float32, 2, 128), (torch.float32, 1, 256),
                                       (torch.float32, 8, 32), (torch.float32, 4, 16), (torch.float32, 8, 8)]
                         + [(dt, h, d) for dt in (torch.float32, torch.bfloat16)
                            for h, d in [(3, 33), (1, 34), (1, 47), (2, 50), (1, 63), (1, 66), (1, 126), (3, 23), (7, 9),
                                         (2, 5), (2, 3), (3, 2), (5, 1)]])
@pytest.mark.parametrize("batched,singles", [(False, False), (True, False), (True, True)])
def test_scores_in_flight_are_those_of_the_scores_call(dtype, H, D, batched, singles):
    """With the same bits in t_j, shipped or formed in flight, every result but the atomically summed one has
    the same bits: the log-sum-exps, the errors and their score gradients take each edge's coefficient."""
    rng, b, _, a_l, a_r = blocks_and_parameters(H, D, sar.SAR_BUILD_SINGLES if singles else sar.SAR_BUILD_NO_SINGLES)
    row = lambda n: torch.from_numpy(rng.standard_normal((n, H, D)).astype(np.float32)).to(dtype).cuda()
    Zs, G = [row(b.n_src(q)) for q in range(2)], row(b.n_dst)
    fwd = gu.gat_fwd_all if batched else gu.gat_fwd_stream
    fw = [fwd(b, Zs[0], Zs, a_l, a_r, SLOPE, fly=fly) for fly in (False, True)]
    assert torch.equal(fw[0].L, fw[1].L)
    assert torch.equal(fw[0].out, fw[1].out)
    g = [gu.gat_bwd(b, Zs[0], Zs, G, a_l, a_r, SLOPE, fw[0], batched, fly=fly) for fly in (False, True)]
    for q in range(2):
        assert torch.equal(g[0].dts[q], g[1].dts[q]), q
        assert torch.equal(g[0].dZs[q], g[1].dZs[q]), q
    b.close()


# wide, few-edge and single-edge sources of every kernel family of the backward pass
@pytest.mark.parametrize("dtype,H,D", [(torch.float32, 4, 64), (torch.bfloat16, 8, 32), (torch.float32, 2, 100),
                                       (torch.bfloat16, 2, 128), (torch.float32, 4, 16), (torch.float32, 1, 47),
                                       (torch.bfloat16, 2, 50), (torch.float32, 2, 3)])
@pytest.mark.parametrize("batched,singles", [(False, False), (True, False), (True, True)])
def test_a_score_of_exactly_zero_takes_the_slope(dtype, H, D, batched, singles):
    """s_i = -t_j, bit for bit, for one in-edge of every destination.  (The derivative at zero is the slope's, the
    oracle's too; no other score of these graphs is within rounding of zero, or the comparison would fail.)"""
    rng, b, want_b, a_l, a_r = blocks_and_parameters(H, D, sar.SAR_BUILD_SINGLES if singles else sar.SAR_BUILD_NO_SINGLES)
    row = lambda n: torch.from_numpy(rng.standard_normal((n, H, D)).astype(np.float32)).to(dtype).cuda()
    Zs, G = [row(b.n_src(q)) for q in range(2)], row(b.n_dst)
    s, ts = gu.gat_scores(Zs[0], Zs, a_l, a_r)
    tied = 0
    for q in (1, 0):                      # the last in-edge of every block, block 0's where a row has both
        has = np.diff(want_b[q].indptr) > 0
        last = want_b[q].indices[want_b[q].indptr[1:][has] - 1]
        s[torch.from_numpy(has).cuda()] = -ts[q][torch.from_numpy(last).long().cuda()]
        tied += has.sum()
    assert tied > b.n_dst / 2
    L, out = torch.empty((b.n_dst, H), device="cuda"), torch.empty((b.n_dst, H, D), dtype=dtype, device="cuda")
    sar.sar_gat_fwd_all(b, Zs, s, ts, a_l, SLOPE, out, L)
    fw = gu.GatOut(out, L, s, ts)
    f64 = gu.host
    want = orc.gat_bwd(want_b, f64(Zs[0]), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE,
                       orc.GatForward(f64(out), f64(L), f64(s), [f64(t) for t in ts]))
    got = gu.gat_bwd(b, Zs[0], Zs, G, a_l, a_r, SLOPE, fw, batched)
    tol = 1e-4 if dtype == torch.float32 else 2e-2
    assert rel_err(f64(got.ds), want.ds) < 1e-4
    for q in range(2):
        assert rel_err(f64(got.dts[q]), want.dt[q]) < 1e-4, q
        assert rel_err(f64(got.dZs[q]), want.dZs[q]) < tol, q
    b.close()


# the infinity is a value that the last two lanes of a head both hold
@pytest.mark.parametrize("H,D,at", [(1, 47, 43), (2, 50, 46), (1, 33, 30), (7, 9, 7), (2, 5, 1)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("fly", [False, True])
def test_a_score_of_minus_infinity_weighs_nothing(H, D, at, dtype, batched, fly):
    """A source whose score is -inf has weight zero: it spoils the column that holds the infinity (0 x inf) in the
    rows that cite it and nothing else."""
    rng, b, want_b, a_l, a_r = blocks_and_parameters(H, D)
    _, without, _, _, _ = blocks_and_parameters(H, D, drop=7)
    Zs = [torch.from_numpy(rng.standard_normal((b.n_src(q), H, D)).astype(np.float32)).to(dtype).cuda() for q in range(2)]
    Zs[0][7, 0, at] = -np.inf * np.sign(a_l[0, at].item())
    s, ts = gu.gat_scores(torch.zeros_like(Zs[0]), Zs, a_l, a_r)
    assert ts[0][7, 0] == -np.inf
    fwd = gu.gat_fwd_all if batched else gu.gat_fwd_stream
    got, want = (fwd(h, torch.zeros_like(Zs[0]), Zs, a_l, a_r, SLOPE, fly=fly) for h in (b, without))
    cited = torch.from_numpy(want_b[0].t_indices[want_b[0].t_indptr[7]:want_b[0].t_indptr[8]]).long().cuda()
    others = torch.ones(b.n_dst, H, D, dtype=torch.bool, device="cuda")
    others[cited, 0, at] = False
    assert cited.numel() and got.out[cited, 0, at].isnan().all()
    rest = got.out[:, 1:][cited] - want.out[:, 1:][cited]      # the other heads still weigh this source
    others[cited, 1:] = False
    tol = 1e-5 if dtype == torch.float32 else 1e-2
    assert torch.isfinite(rest).all()
    assert torch.allclose(got.out[others].float(), want.out[others].float(), rtol=tol, atol=tol)
    assert torch.allclose(got.L[:, 0], want.L[:, 0], rtol=1e-5, atol=1e-5)
    b.close()
    without.close()
