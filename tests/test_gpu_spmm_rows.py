"""Sum / mean aggregation of rows whose width is no whole number of 16-byte pieces, and of the rows with
fewer than 8 edges that share a wavefront: every width at which the lanes of a row change."""
import numpy as np
import pytest
import torch

from oracle import sar_oracle as orc
from paper_2111_06483_amd import sar
from tests import gpu_util as gu
from tests.helpers import rel_err, tiny_graph

pytestmark = pytest.mark.gpu
f64 = lambda t: t.to(torch.float64).cpu().numpy()


@pytest.mark.parametrize("F", [3, 4, 5, 9, 15, 17, 31, 47, 65, 127, 129, 255, 257, 511, 513])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("E", [3_000, 14_000])          # nearly all rows below 8 edges; about half of them
def test_rows(F, dtype, E):
    rng = np.random.default_rng(F)
    src, dst, part = tiny_graph(rng, 1_500, E, 3, simple=False)
    want_b, _ = orc.build_blocks(src, dst, part, 3, 1)
    row = lambda n: torch.from_numpy(rng.standard_normal((n, F)).astype(np.float32)).to(dtype).cuda()
    for flags in (0, sar.SAR_BUILD_COMPACT):
        b = gu.build_blocks(src, dst, part, 3, 1, flags=sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | flags)
        Zs, G = [row(w.n_src) for w in want_b], row(b.n_dst)
        want = orc.spmm(want_b, [f64(z) for z in Zs], True)
        tol = 1e-5 if dtype == torch.float32 else 1e-2
        assert rel_err(f64(gu.spmm_stream(b, Zs, True)), want) < tol
        assert rel_err(f64(gu.spmm_all(b, Zs, True)), want) < tol
        want_d = orc.spmm_bwd(want_b, f64(G), True)
        dZs = [torch.full((b.n_err_rows(q), F), float("nan"), dtype=dtype, device="cuda") for q in range(3)]
        dZb = [torch.full_like(d, float("nan")) for d in dZs]
        sar.sar_spmm_bwd_all(b, G, True, dZs)
        for q in range(3):
            sar.sar_spmm_bwd_block(b, q, G, True, dZb[q])
            keep = np.diff(want_b[q].t_indptr) > 0 if flags else slice(None)
            for got in (dZs[q], dZb[q]):
                assert rel_err(f64(got), want_d[q][keep]) < tol, q
        b.close()


# rows wider than a wavefront in launches of even width, the last of which would be left with one to three (fp32) or
# one to seven (bf16) values, or just has a piece
@pytest.mark.parametrize("dtype,F", [(torch.float32, 16129), (torch.float32, 16130), (torch.float32, 16131),
                                     (torch.float32, 16132), (torch.float32, 16385), (torch.bfloat16, 32257),
                                     (torch.bfloat16, 32263), (torch.bfloat16, 32264)])
def test_last_column_range(dtype, F):
    rng = np.random.default_rng(F)
    src, dst, part = tiny_graph(rng, 60, 400, 2, simple=False)
    want_b, _ = orc.build_blocks(src, dst, part, 2, 1)
    b = gu.build_blocks(src, dst, part, 2, 1)
    row = lambda n: torch.from_numpy(rng.standard_normal((n, F)).astype(np.float32)).to(dtype).cuda()
    Zs, G = [row(w.n_src) for w in want_b], row(b.n_dst)
    want = orc.spmm(want_b, [f64(z) for z in Zs], True)
    tol = 1e-5 if dtype == torch.float32 else 1e-2
    assert rel_err(f64(gu.spmm_stream(b, Zs, True)), want) < tol
    assert rel_err(f64(gu.spmm_all(b, Zs, True)), want) < tol
    want_d = orc.spmm_bwd(want_b, f64(G), True)
    dZs = [torch.full_like(z, float("nan")) for z in Zs]
    sar.sar_spmm_bwd_all(b, G, True, dZs)
    for q in range(2):
        assert rel_err(f64(dZs[q]), want_d[q]) < tol, q
    b.close()
