"""The backward pass of a small call is one launch (wide sources, sources of few edges and single-edge sources together); a
larger one takes a launch for each.  Both sides of that line, in the three lane layouts that have it, against the
oracle; the tolerances are those of the types (fp32 sums of fp32 rows; one bf16 rounding of the results)."""
import numpy as np
import pytest
import torch

from oracle import sar_oracle as orc
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2111_06483_amd import sar
    from tests import gpu_util as gu

TOL = {torch.float32: 1e-4, torch.bfloat16: 2e-2}
SLOPE = 0.2


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this process")
    sar.lib()


def graph(seed, n_dst, per_block, P):
    """Partition 0 holds the destinations; a source elsewhere has 0, 1, 2..7 or 8..20 edges.  Every destination cites itself
    and its neighbour."""
    rng = np.random.default_rng(seed)
    n = (P - 1) * per_block
    k = np.choose(rng.integers(0, 4, n), [np.zeros(n, int), np.ones(n, int), rng.integers(2, 8, n), rng.integers(8, 21, n)])
    first = rng.integers(0, n_dst, n)
    src = np.repeat(np.arange(n_dst, n_dst + n), k)
    at = np.arange(len(src)) - np.repeat(np.cumsum(k) - k, k)
    dst = (np.repeat(first, k) + 7 * at) % n_dst             # 20 steps of 7 stay under n_dst: no edge twice
    own = np.arange(n_dst)
    src = np.concatenate([src, own, own])
    dst = np.concatenate([dst, own, (own + 1) % n_dst])
    part = np.concatenate([np.zeros(n_dst, np.int32), np.repeat(np.arange(1, P), per_block).astype(np.int32)])
    return src.astype(np.int64), dst.astype(np.int64), part, rng


# exact lanes, padded lanes, two and more rows to a wavefront with a list of singles and without one
@pytest.mark.parametrize("dtype,H,D,flags", [(torch.float32, 8, 32, 0), (torch.bfloat16, 4, 64, 0), (torch.bfloat16, 2, 100, 0),
                                             (torch.float32, 4, 32, 16), (torch.bfloat16, 4, 16, 0)])
@pytest.mark.parametrize("compact", [False, True])
@pytest.mark.parametrize("per_block", [1, 40, 700, 24000])
def test_one_launch_and_several(dtype, H, D, flags, compact, per_block):
    P, n_dst = 3, 150
    src, dst, part, rng = graph(5, n_dst, per_block, P)
    w_b, _ = orc.build_blocks(src, dst, part, P, 0)
    single = sar.SAR_BUILD_NO_SINGLES if flags else sar.SAR_BUILD_SINGLES
    b = gu.build_blocks(src, dst, part, P, 0, flags=3 | single | (sar.SAR_BUILD_COMPACT if compact else 0))
    Zs = [torch.from_numpy(rng.standard_normal((w.n_src, H, D)).astype(np.float32)).to(dtype).cuda() for w in w_b]
    bound = np.sqrt(6.0 / (D + 1))
    a_l, a_r = (torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda() for _ in range(2))
    G = torch.from_numpy(rng.standard_normal((n_dst, H, D)).astype(np.float32)).to(dtype).cuda()
    f64 = lambda t: t.to(torch.float64).cpu().numpy()
    Z64 = [f64(z) for z in Zs]
    wf = orc.gat_fwd(w_b, Z64[0], Z64, f64(a_l), f64(a_r), SLOPE)
    wb = orc.gat_bwd(w_b, Z64[0], Z64, f64(G), f64(a_l), f64(a_r), SLOPE, wf)
    fw = gu.gat_fwd_all(b, Zs[0], Zs, a_l, a_r, SLOPE)
    rows = [np.flatnonzero(np.diff(w.t_indptr) > 0) if compact else np.arange(w.n_src) for w in w_b]
    work = torch.empty(sar.sar_gat_workspace_bytes(n_dst, 0, H, D) // 4, dtype=torch.float32, device="cuda")
    rec = torch.empty((n_dst, H, 4), dtype=torch.float32, device="cuda")
    ds = torch.empty((n_dst, H), dtype=torch.float32, device="cuda")
    sar.sar_gat_bwd_begin(G, fw.out, fw.s, fw.L, rec, ds)
    da_l = torch.zeros((H, D), dtype=torch.float32, device="cuda")
    dZs = [torch.full((len(r), H, D), float("nan"), dtype=dtype, device="cuda") for r in rows]
    dts = [torch.full((len(r), H), float("nan"), dtype=torch.float32, device="cuda") for r in rows]
    sar.sar_gat_bwd_all(b, Zs, G, None, rec, a_l, SLOPE, dZs, dts, ds, da_l, work)
    tol = TOL[dtype]
    # Against the largest value of all blocks: a block may be one row, and an edge's share of dt is alpha (<G, Z> - <G, out>)
    # with `out` rounded to the rows' type, an error of 2^-9 alpha |G| |out| in bf16 however small the difference is.
    together = lambda xs: np.concatenate([f64(x) if torch.is_tensor(x) else x for x in xs])
    assert rel_err(together(dZs), together([wb.dZs[q][rows[q]] for q in range(P)])) < tol
    assert rel_err(together(dts), together([wb.dt[q][rows[q]] for q in range(P)])) < tol
    assert rel_err(f64(ds), wb.ds) < tol
    assert rel_err(f64(da_l), wb.da_l) < tol
    b.close()
