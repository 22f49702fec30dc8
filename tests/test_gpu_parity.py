"""Parity of the HIP path (through the C ABI) with the CPU oracle, element by element.

Tolerances: bit-exact for the block index; tensor-scale relative
error max|a-b|/max|b| <= 1e-4 for fp32 tensors; <= 2e-2 for bf16-stored
tensors with fp32 accumulation.  The oracle always runs in fp64 on the same
(already rounded) inputs.
"""
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
    sar.lib()   # raises if the HIP library is missing: no fallback


def make_graph(seed, N, E, P, hubs=True, simple=True, empty_block=None):
    """Random directed graph with a heavy destination, a heavy source and ragged sizes."""
    rng = np.random.default_rng(seed)
    src = rng.integers(0, N, size=E)
    dst = rng.integers(0, N, size=E)
    part = rng.integers(0, P, size=N).astype(np.int32)
    part[:P] = np.arange(P)
    if hubs:
        k = min(N, 1500)
        hub_dst = int(np.flatnonzero(part == 0)[0])
        hub_src = int(np.flatnonzero(part == P - 1)[-1])
        src = np.concatenate([src, rng.choice(N, k, replace=False), np.full(k, hub_src)])
        dst = np.concatenate([dst, np.full(k, hub_dst), rng.choice(N, k, replace=False)])
    if empty_block is not None:
        keep = part[src] != empty_block
        src, dst = src[keep], dst[keep]
    if simple:
        key = np.unique(dst.astype(np.int64) * N + src)
        dst, src = key // N, key % N
    return src.astype(np.int64), dst.astype(np.int64), part, rng


def feats(rng, n, F, dtype, scale=1.0):
    x = torch.from_numpy((rng.standard_normal((n, F)) * scale).astype(np.float32)).to(dtype)
    return x


def f64(t):
    return t.to(torch.float64).cpu().numpy()


# ------------------------------------------------------------------ builder

def expected_long(deg):
    """Rows shared by a workgroup: those of at least 128, 256 or 512 edges, the lowest threshold
    that leaves them at most a sixteenth of the rows with edges (or 256 rows)."""
    n_rows = int(np.sum(deg > 0))
    for t in (128, 256):
        if int(np.sum(deg >= t)) <= max(256, n_rows // 16):
            return int(np.sum(deg >= t))
    return int(np.sum(deg >= 512))


@pytest.mark.parametrize("idx_dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("N,E,P,p,simple", [(3000, 40000, 3, 0, True), (5000, 30000, 7, 6, False),
                                            (257, 900, 1, 0, False), (70000, 150000, 16, 3, True)])
def test_builder_bit_exact(N, E, P, p, simple, idx_dtype):
    src, dst, part, _ = make_graph(1, N, E, P, simple=simple, empty_block=(1 if P > 2 else None))
    want, want_deg = orc.build_blocks(src, dst, part, P, p)
    b = gu.build_blocks(src, dst, part, P, p, idx_dtype=idx_dtype)
    assert b.P == P and b.n_dst == want[0].n_dst
    assert np.array_equal(sar.sar_blocks_degree(b).cpu().numpy(), want_deg)
    for q in range(P):
        v = gu.view_arrays(b, q)
        w = want[q]
        assert (v["n_dst"], v["n_src"], v["nnz"]) == (w.n_dst, w.n_src, w.nnz)
        assert np.array_equal(v["indptr"], w.indptr.astype(np.int32))
        assert np.array_equal(v["indices"], w.indices)
        assert np.array_equal(v["t_indptr"], w.t_indptr.astype(np.int32))
        assert np.array_equal(v["t_indices"], w.t_indices)
        # launch lists: exactly the non-empty rows, longest degree class first
        deg_q = np.diff(w.indptr)
        assert sorted(v["rows"].tolist()) == np.flatnonzero(deg_q > 0).tolist()
        cls = np.floor(np.log2(np.maximum(deg_q[v["rows"]], 1))).astype(int)
        assert np.all(np.diff(cls) <= 0)
        assert v["n_long"] == expected_long(deg_q)
        tdeg = np.diff(w.t_indptr)
        assert sorted(v["t_rows"].tolist()) == np.flatnonzero(tdeg > 0).tolist()
        assert np.array_equal(v["touched"], np.flatnonzero(tdeg > 0).astype(np.int32))
        assert v["n_t_long"] == expected_long(tdeg)
    b.close()


def test_builder_rejects_bad_input():
    src, dst, part, _ = make_graph(2, 500, 2000, 2, hubs=False)
    bad = src.copy()
    bad[7] = 500
    with pytest.raises(sar.SarError) as e:
        gu.build_blocks(bad, dst, part, 2, 0)
    assert e.value.code == sar.SAR_ERR_INVALID_ARG
    badp = part.copy()
    badp[3] = 2
    with pytest.raises(sar.SarError):
        gu.build_blocks(src, dst, badp, 2, 0)
    with pytest.raises(sar.SarError):
        gu.build_blocks(src, dst, part, 2, 2)


def test_wrap_equals_build():
    src, dst, part, rng = make_graph(3, 2000, 20000, 3)
    want, _ = orc.build_blocks(src, dst, part, 3, 1)
    indptr = [gu.dev(w.indptr, torch.int32) for w in want]
    indices = [gu.dev(w.indices, torch.int32) for w in want]
    b = sar.sar_blocks_wrap(want[0].n_dst, [w.n_src for w in want], indptr, indices)
    for q in range(3):
        v = gu.view_arrays(b, q)
        assert np.array_equal(v["t_indptr"], want[q].t_indptr.astype(np.int32))
        assert np.array_equal(v["t_indices"], want[q].t_indices)
    Zs = [feats(rng, w.n_src, 32, torch.float32).cuda() for w in want]
    got = gu.spmm_all(b, Zs, True)
    assert rel_err(f64(got), orc.spmm(want, [f64(z) for z in Zs], True)) < 1e-4
    b.close()


# --------------------------------------------------------------------- spmm

@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [8, 64, 200, 256, 800, 1032, 50, 7, 130, 33])
@pytest.mark.parametrize("mean", [False, True])
def test_spmm_parity(dtype, F, mean):
    src, dst, part, rng = make_graph(4, 3000, 40000, 3, simple=False)
    want_b, deg = orc.build_blocks(src, dst, part, 3, 0)
    b = gu.build_blocks(src, dst, part, 3, 0)
    Zs = [feats(rng, w.n_src, F, dtype).cuda() for w in want_b]
    want = orc.spmm(want_b, [f64(z) for z in Zs], mean)
    assert rel_err(f64(gu.spmm_stream(b, Zs, mean)), want) < TOL[dtype]
    assert rel_err(f64(gu.spmm_all(b, Zs, mean)), want) < TOL[dtype]
    # case 1 backward
    G = feats(rng, b.n_dst, F, dtype).cuda()
    want_d = orc.spmm_bwd(want_b, f64(G), mean)
    for q in range(3):
        dZ = torch.full(Zs[q].shape, float("nan"), dtype=dtype, device="cuda")
        sar.sar_spmm_bwd_block(b, q, G, mean, dZ)
        assert rel_err(f64(dZ), want_d[q]) < TOL[dtype]
    dZs = [torch.full(z.shape, float("nan"), dtype=dtype, device="cuda") for z in Zs]
    sar.sar_spmm_bwd_all(b, G, mean, dZs)
    for q in range(3):
        assert rel_err(f64(dZs[q]), want_d[q]) < TOL[dtype]
    b.close()


def test_spmm_all_ones_gives_degree_exactly():
    src, dst, part, rng = make_graph(5, 3000, 40000, 4, simple=False)
    b = gu.build_blocks(src, dst, part, 4, 2)
    _, deg = orc.build_blocks(src, dst, part, 4, 2)
    Zs = [torch.ones((b.view(q).n_src, 16), device="cuda") for q in range(4)]
    out = gu.spmm_all(b, Zs, False).cpu().numpy()
    assert np.array_equal(out, np.repeat(deg[:, None], 16, 1).astype(np.float32))
    b.close()


# ---------------------------------------------------------------------- GAT

def gat_case(seed, N, E, P, p, H, D, dtype, scale=1.0, simple=True, empty_block=None):
    src, dst, part, rng = make_graph(seed, N, E, P, simple=simple, empty_block=empty_block)
    want_b, deg = orc.build_blocks(src, dst, part, P, p)
    b = gu.build_blocks(src, dst, part, P, p)
    F = H * D
    Zs = [feats(rng, w.n_src, F, dtype, scale).cuda().reshape(-1, H, D) for w in want_b]
    Zdst = feats(rng, b.n_dst, F, dtype, scale).cuda().reshape(-1, H, D)
    bound = np.sqrt(6.0 / (D + 1))      # Xavier-uniform, as in the configurations: scores of O(1)
    a_l = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    a_r = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    G = feats(rng, b.n_dst, F, dtype).cuda().reshape(-1, H, D)
    return b, want_b, deg, Zdst, Zs, a_l, a_r, G


def check_fwd(got, want, deg, dtype):
    tol = TOL[dtype]
    assert rel_err(f64(got.out), want.out) < tol
    Lg = f64(got.L)
    has = deg > 0
    assert np.all(np.isneginf(Lg[~has])) and np.all(f64(got.out)[~has] == 0)
    assert rel_err(Lg[has], want.L[has]) < 1e-4          # L is fp32 state in both dtypes
    assert rel_err(f64(got.s), want.s) < 1e-4
    for tg, tw in zip(got.t, want.t):
        assert rel_err(f64(tg), tw) < 1e-4


# (heads, head width): every lane mapping of the generic kernels, every head width of the F = 256
# kernels, non-power-of-two heads, and rows wider than 1 KiB (processed as groups of heads)
SHAPES = [(4, 16), (1, 4), (4, 64), (8, 32), (2, 100), (3, 12), (1, 256), (2, 128), (16, 16),
          (8, 100), (8, 64), (3, 200), (2, 256), (1, 512),      # the last: the widest head of each row type
          # padded geometry with idle lanes: half-filled head groups, 8 lanes per head, and the sparse
          # single-launch layers whose backward pass alone takes the specialised kernels
          (4, 32), (2, 64), (1, 128), (16, 32), (1, 100), (6, 36), (8, 16), (8, 8), (2, 32), (1, 64), (2, 16),
          (8, 20), (12, 16),
          # head counts that leave whole head groups of the padded geometry without a head
          (3, 64), (6, 32), (5, 8), (7, 8), (3, 32), (5, 40),
          # head widths that are not whole 16-byte pieces: lanes move 8, 4 or 2 bytes
          (3, 10), (2, 50), (4, 12), (5, 7), (2, 63), (1, 126), (6, 36)]


def supported(dtype, D):
    """Lanes move the largest piece of 16, 8, 4 (bf16: 2) bytes that divides the head; a head fits 64 lanes."""
    piece = 4 if dtype == torch.float32 else 8
    while D % piece:
        piece //= 2
    return D // piece <= 64


CASES = [(dt, H, D) for dt in (torch.float32, torch.bfloat16) for H, D in SHAPES if supported(dt, D)]


@pytest.mark.parametrize("dtype,H,D", CASES)
def test_gat_forward_parity(dtype, H, D):
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(6, 3000, 40000, 3, 0, H, D, dtype, simple=False)
    want = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    states = []
    check_fwd(gu.gat_fwd_stream(b, Zdst, Zs, a_l, a_r, SLOPE, states=states), want, deg, dtype)
    check_fwd(gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE), want, deg, dtype)
    # source score halves formed inside the kernels instead of read from tq
    check_fwd(gu.gat_fwd_stream(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True), want, deg, dtype)
    check_fwd(gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True), want, deg, dtype)
    # the carried state after block k represents Eq. 3 restricted to blocks 0..k
    for k, (m, l, acc) in enumerate(states[:-1]):
        part = orc.gat_fwd(want_b[:k + 1], f64(Zdst), [f64(z) for z in Zs[:k + 1]], f64(a_l), f64(a_r), SLOPE)
        seen = l > 0
        assert np.array_equal(seen, np.isfinite(part.L))
        got = np.where(seen[:, :, None], acc / np.where(seen, l, 1)[:, :, None], 0)
        assert rel_err(got, part.out) < 1e-4
        assert rel_err((m + np.log(np.where(seen, l, 1)))[seen], part.L[seen]) < 1e-4
    b.close()


@pytest.mark.parametrize("dtype,H,D", CASES)
@pytest.mark.parametrize("batched,fly", [(False, False), (True, False), (True, True), (False, True)])
def test_gat_backward_parity(dtype, H, D, batched, fly):
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(7, 3000, 40000, 3, 1, H, D, dtype)
    wf = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    wb = orc.gat_bwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE, wf)
    fw = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE)
    g = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, fw, batched, fly=fly)
    tol = TOL[dtype]
    for q in range(b.P):
        assert rel_err(f64(g.dZs[q]), wb.dZs[q]) < tol, q
        assert rel_err(f64(g.dts[q]), wb.dt[q]) < tol, q
    assert rel_err(f64(g.ds), wb.ds) < tol
    assert rel_err(f64(g.dZdst), wb.dZdst) < tol
    assert rel_err(f64(g.da_l), wb.da_l) < tol
    assert rel_err(f64(g.da_r), wb.da_r) < tol
    # the local block's error added into the destination-side error in the same pass
    g2 = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, fw, batched, fly=fly, dZadd=G)
    assert rel_err(f64(g2.dZdst), wb.dZdst + f64(G)) < tol
    b.close()


@pytest.mark.parametrize("dtype,H,D", [(torch.float32, 4, 64), (torch.bfloat16, 8, 32), (torch.float32, 2, 100),
                                       (torch.bfloat16, 4, 32), (torch.float32, 3, 10), (torch.bfloat16, 5, 40)])
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("full_height", [False, True])
def test_backward_without_the_dt_output(dtype, H, D, batched, full_height):
    """dt_q is an intermediate of the backward kernels; a call that does not ask for it (dtq NULL) gives
    the same dZ_q and da_l bit for bit (neither involves an atomic) and the same ds up to the order
    of its atomic sums.  Full-height handles also write the zero rows of the sources without an edge."""
    src, dst, part, rng = make_graph(23, 3000, 9000, 3, empty_block=None)
    flags = sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | (0 if full_height else sar.SAR_BUILD_COMPACT)
    want_b, _ = orc.build_blocks(src, dst, part, 3, 1)
    b = gu.build_blocks(src, dst, part, 3, 1, flags=flags)
    rows = [w.n_src if full_height else int(np.count_nonzero(np.diff(w.t_indptr))) for w in want_b]
    F = H * D
    Zs = [feats(rng, w.n_src, F, dtype).cuda().reshape(-1, H, D) for w in want_b]
    Zdst = Zs[1]
    bound = np.sqrt(6.0 / (D + 1))
    a_l = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    a_r = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    G = feats(rng, b.n_dst, F, dtype).cuda().reshape(-1, H, D)
    fw = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True)
    n = b.n_dst
    work = torch.empty(sar.sar_gat_workspace_bytes(n, 0, H, D) // 4, dtype=torch.float32, device="cuda")
    res = []
    for store_dt in (True, False):
        rec = torch.empty((n, H, 4), dtype=torch.float32, device="cuda")
        ds = torch.empty((n, H), dtype=torch.float32, device="cuda")
        sar.sar_gat_bwd_begin(G, fw.out, fw.s, fw.L, rec, ds)
        da_l = torch.zeros((H, D), dtype=torch.float32, device="cuda")
        dZs = [torch.full((r, H, D), float("nan"), dtype=dtype, device="cuda") for r in rows]
        dts = [torch.full((r, H), float("nan"), dtype=torch.float32, device="cuda") for r in rows] if store_dt else None
        if batched:
            sar.sar_gat_bwd_all(b, Zs, G, None, rec, a_l, SLOPE, dZs, dts, ds, da_l, work)
        else:
            for q in range(3):
                sar.sar_gat_bwd_block(b, q, Zs[q], G, None, rec, a_l, SLOPE, dZs[q], dts[q] if store_dt else None,
                                      ds, da_l, work)
        res.append((dZs, dts, ds, da_l))
    (dZ1, dt1, ds1, da1), (dZ0, _, ds0, da0) = res
    for q in range(3):
        assert not torch.isnan(dZ0[q].float()).any() and not torch.isnan(dt1[q]).any()
        assert torch.equal(dZ0[q], dZ1[q]), q
    assert torch.equal(da0, da1)
    assert rel_err(f64(ds0), f64(ds1)) < 1e-5
    b.close()


@pytest.mark.parametrize("dtype,H,D", [(torch.float32, 4, 64), (torch.bfloat16, 8, 32), (torch.float32, 16, 16),
                                       (torch.bfloat16, 1, 256), (torch.float32, 2, 128)])
@pytest.mark.parametrize("n_src,degs", [(1, (3,)), (5, (1,)), (6, (7,)), (203, (1, 2, 3, 4, 5, 6, 7)), (66, (2, 7)),
                                        (1027, (1, 1, 1, 2, 6))])
def test_backward_sources_of_few_edges(dtype, H, D, n_src, degs):
    """Sources of 1..7 edges only (the kernel that takes several sources per wavefront): every
    degree, groups whose sources differ in degree, counts that do not fill the last group, one
    source alone.  Partition 1 holds the sources, partition 0 the 40 destinations (each of which
    also cites two others, so the local block has few-edge sources too)."""
    rng = np.random.default_rng(100 * n_src + len(degs))
    n_dst = 40
    src, dst = [], []
    for j in range(n_src):
        k = degs[j % len(degs)]
        src += [n_dst + j] * k
        dst += rng.choice(n_dst, k, replace=False).tolist()
    for j in range(n_dst):      # every destination has two local in-edges: no coefficient is exactly 1
        src += [j, j]
        dst += [(j + 1) % n_dst, (j + 7) % n_dst]
    src, dst = np.array(src, dtype=np.int64), np.array(dst, dtype=np.int64)
    part = np.concatenate([np.zeros(n_dst, np.int32), np.ones(n_src, np.int32)])
    want_b, deg = orc.build_blocks(src, dst, part, 2, 0)
    assert max(int(np.diff(w.t_indptr).max()) for w in want_b) < 8
    b = gu.build_blocks(src, dst, part, 2, 0)
    F = H * D
    Zs = [feats(rng, w.n_src, F, dtype).cuda().reshape(-1, H, D) for w in want_b]
    Zdst = feats(rng, n_dst, F, dtype).cuda().reshape(-1, H, D)
    bound = np.sqrt(6.0 / (D + 1))
    a_l = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    a_r = torch.from_numpy(rng.uniform(-bound, bound, (H, D)).astype(np.float32)).cuda()
    G = feats(rng, n_dst, F, dtype).cuda().reshape(-1, H, D)
    wf = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    wb = orc.gat_bwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE, wf)
    fw = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE)
    tol = TOL[dtype]
    for batched in (False, True):
        for fly in (False, True):
            g = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, fw, batched, fly=fly)
            for q in range(2):
                assert rel_err(f64(g.dZs[q]), wb.dZs[q]) < tol, (batched, fly, q)
                assert rel_err(f64(g.dts[q]), wb.dt[q]) < tol, (batched, fly, q)
            assert rel_err(f64(g.ds), wb.ds) < tol
            assert rel_err(f64(g.da_l), wb.da_l) < tol
    b.close()


def test_gat_edge_cases():
    """Empty block, single block, destinations without edges, block order, big scores."""
    H, D = 4, 16
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(8, 2000, 6000, 4, 2, H, D, torch.float32,
                                                     scale=40.0, empty_block=1)
    assert want_b[1].nnz == 0 and (deg == 0).any()
    want = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    assert np.abs(want.s).max() > 100          # exp() of these overflows fp32 without the running max
    got = gu.gat_fwd_stream(b, Zdst, Zs, a_l, a_r, SLOPE)
    check_fwd(got, want, deg, torch.float32)
    assert torch.isfinite(got.out).all()
    perm = gu.gat_fwd_stream(b, Zdst, Zs, a_l, a_r, SLOPE, order=[3, 1, 0, 2])
    assert rel_err(f64(perm.out), want.out) < 1e-4
    allb = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE)
    check_fwd(allb, want, deg, torch.float32)
    wb = orc.gat_bwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE, want)
    for batched in (False, True):
        g = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, allb, batched)
        for q in range(4):
            assert rel_err(f64(g.dZs[q]), wb.dZs[q]) < 1e-4
        assert torch.all(g.dZs[1] == 0)
        assert rel_err(f64(g.da_l), wb.da_l) < 1e-4 and rel_err(f64(g.da_r), wb.da_r) < 1e-4
        assert rel_err(f64(g.dZdst), wb.dZdst) < 1e-4
    b.close()


def test_gat_zero_attention_equals_mean_kernel():
    """a = 0 makes attention uniform: the GAT kernels must agree with the SpMM-mean kernel."""
    H, D = 2, 32
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(9, 3000, 30000, 3, 0, H, D, torch.float32)
    zero = torch.zeros_like(a_l)
    got = gu.gat_fwd_all(b, Zdst, Zs, zero, zero, SLOPE)
    mean = gu.spmm_all(b, [z.reshape(-1, H * D) for z in Zs], True)
    assert rel_err(f64(got.out).reshape(-1, H * D), f64(mean)) < 1e-5
    b.close()


def test_config1_full():
    """Configuration 1: 4096-node Chung-Lu graph, self-loops, 1 block, 64 -> 4 x 16, fp32."""
    from paper_2111_06483_amd import synth
    w = synth.make_workload("cfg1")
    members = w.members(0)
    X = synth.normal_rows(2, members, w.f_in)
    W, a_l, a_r = synth.gat_params(3, w.f_in, w.H, w.D)
    G = synth.normal_rows(4, members, w.H * w.D).reshape(-1, w.H, w.D)
    want_b, deg = orc.build_blocks(w.src.numpy(), w.dst.numpy(), w.part.numpy(), 1, 0)
    res = orc.gat_layer(want_b, f64(X), [f64(X)], f64(W), f64(a_l), f64(a_r), w.slope, f64(G))

    b = sar.sar_blocks_build(w.src.cuda(), w.dst.cuda(), w.part.cuda(), 1, 0)
    v = gu.view_arrays(b, 0)
    assert np.array_equal(v["indptr"], want_b[0].indptr.astype(np.int32))
    assert np.array_equal(v["indices"], want_b[0].indices)
    Xd, Wd, ald, ard, Gd = X.cuda(), W.cuda(), a_l.cuda(), a_r.cuda(), G.cuda()
    Z, s, t = gu.linear_fwd(Xd, Wd, ard, ald)
    assert rel_err(f64(Z), res.Zdst.reshape(Z.shape)) < 1e-4
    Z3 = Z.reshape(-1, w.H, w.D)
    for fwd in (gu.gat_fwd_stream, gu.gat_fwd_all):
        fw = fwd(b, Z3, [Z3], ald, ard, w.slope)
        check_fwd(fw, res.fwd, deg, torch.float32)
    for batched in (False, True):
        g = gu.gat_bwd(b, Z3, [Z3], Gd, ald, ard, w.slope, fw, batched)
        assert rel_err(f64(g.dZs[0]), res.bwd.dZs[0]) < 1e-4
        assert rel_err(f64(g.dZdst), res.bwd.dZdst) < 1e-4
        assert rel_err(f64(g.da_l), res.bwd.da_l) < 1e-4
        assert rel_err(f64(g.da_r), res.bwd.da_r) < 1e-4
    # the transform's backward: destination rows and the (local) source block add up in dW
    dW = torch.zeros_like(Wd)
    dXd = gu.linear_bwd(Xd, g.dZdst, Wd, dW)
    dXs = gu.linear_bwd(Xd, g.dZs[0], Wd, dW)
    assert rel_err(f64(dW), res.dW) < 1e-4
    assert rel_err(f64(dXd), res.dXdst) < 1e-4
    assert rel_err(f64(dXs), res.dXs[0]) < 1e-4
    b.close()


# ------------------------------------------------------------------- linear

@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,K,F", [(1000, 100, 256), (333, 64, 64), (4097, 128, 256), (130, 256, 40),
                                   (2050, 104, 800), (517, 36, 200), (700, 602, 64), (31, 8, 8), (77, 30, 50)])
def test_linear_parity(dtype, n, K, F):
    rng = np.random.default_rng(10)
    X = feats(rng, n, K, dtype).cuda()
    W = torch.from_numpy((rng.standard_normal((K, F)) * 0.1).astype(np.float32)).cuda()
    dZ = feats(rng, n, F, dtype).cuda()
    Z, _, _ = gu.linear_fwd(X, W)
    assert rel_err(f64(Z), orc.linear_fwd(f64(X), f64(W))) < (1e-4 if dtype == torch.float32 else 2e-2)
    dW = torch.zeros_like(W)
    dX = gu.linear_bwd(X, dZ, W, dW)
    want_dW, want_dX = orc.linear_bwd(f64(X), f64(dZ), f64(W))
    assert rel_err(f64(dW), want_dW) < 1e-4      # dW is fp32 in both storage types
    assert rel_err(f64(dX), want_dX) < TOL[dtype]
    # accumulates
    gu.linear_bwd(X, dZ, W, dW)
    assert rel_err(f64(dW), 2 * want_dW) < 1e-4


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,K,H,D", [(1500, 100, 4, 64), (700, 128, 8, 32), (333, 64, 1, 256), (260, 40, 2, 100),
                                     (90, 30, 3, 24), (300, 64, 20, 8), (500, 602, 4, 16),
                                     # two column slabs: heads inside a slab, and a head across the boundary
                                     (700, 256, 8, 32), (300, 256, 2, 104), (300, 256, 3, 88)])
def test_linear_scores_parity(dtype, n, K, H, D):
    """The two score projections of Eq. 3 that come out of the transform: s = a1 . z and
    t = a2 . z per head, against the oracle's scores of its own fp64 Z = X W."""
    rng = np.random.default_rng(13)
    F = H * D
    X = feats(rng, n, K, dtype).cuda()
    W = torch.from_numpy((rng.standard_normal((K, F)) * 0.1).astype(np.float32)).cuda()
    a1 = torch.from_numpy(rng.standard_normal((H, D)).astype(np.float32)).cuda()
    a2 = torch.from_numpy(rng.standard_normal((H, D)).astype(np.float32)).cuda()
    Z, s, t = gu.linear_fwd(X, W, a1, a2)
    wantZ = orc.linear_fwd(f64(X), f64(W))
    tol = 1e-4 if dtype == torch.float32 else 2e-2
    assert rel_err(f64(Z), wantZ) < tol
    assert rel_err(f64(s), orc.gat_scores(wantZ.reshape(n, H, D), f64(a1))) < tol
    assert rel_err(f64(t), orc.gat_scores(wantZ.reshape(n, H, D), f64(a2))) < tol
    # one projection only
    _, s_only, _ = gu.linear_fwd(X, W, a1, None)
    assert torch.equal(s_only, s)


# ------------------------------------------------------- streams, determinism, errors

def test_stream_argument_and_determinism():
    """Launches go to the stream they are given; everything except the atomically accumulated
    ds (and what is derived from it) is bitwise reproducible."""
    H, D = 4, 64
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(11, 3000, 40000, 3, 0, H, D, torch.float32)
    ref = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        again = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True)
    side.synchronize()
    assert torch.equal(ref.out, again.out) and torch.equal(ref.L, again.L)
    g1 = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, ref, True, fly=True)
    with torch.cuda.stream(side):
        g2 = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, ref, True, fly=True)
    side.synchronize()
    for q in range(b.P):
        assert torch.equal(g1.dZs[q], g2.dZs[q]) and torch.equal(g1.dts[q], g2.dts[q])
    assert torch.equal(g1.da_l, g2.da_l)
    assert rel_err(f64(g2.ds), f64(g1.ds)) < 1e-5       # atomics: order may differ, values agree
    b.close()


def test_error_paths():
    src, dst, part, rng = make_graph(12, 1000, 8000, 2, hubs=False)
    H, D = 2, 16
    b0 = gu.build_blocks(src, dst, part, 2, 0, flags=0)          # no transpose, no all-blocks index
    n = b0.n_dst
    Zs = [feats(rng, b0.view(q).n_src, H * D, torch.float32).cuda().reshape(-1, H, D) for q in range(2)]
    a = torch.zeros((H, D), device="cuda")
    s = torch.zeros((n, H), device="cuda")
    out = torch.empty((n, H, D), device="cuda")
    L = torch.empty((n, H), device="cuda")
    with pytest.raises(sar.SarError) as e:
        sar.sar_gat_fwd_all(b0, Zs, s, None, a, SLOPE, out, L)
    assert e.value.code == sar.SAR_ERR_STATE
    rec = torch.zeros((n, H, 4), device="cuda")
    ds = torch.zeros((n, H), device="cuda")
    work = torch.empty(sar.sar_gat_workspace_bytes(n, n, H, D) // 4, device="cuda")
    with pytest.raises(sar.SarError) as e:
        sar.sar_gat_bwd_block(b0, 0, Zs[0], out, None, rec, a, SLOPE, torch.empty_like(Zs[0]),
                              torch.empty((Zs[0].shape[0], H), device="cuda"), ds, torch.zeros_like(a), work)
    assert e.value.code == sar.SAR_ERR_STATE
    b0.close()
    b = gu.build_blocks(src, dst, part, 2, 0)
    with pytest.raises(sar.SarError) as e:      # scratch too small
        sar.sar_gat_bwd_block(b, 0, Zs[0], out, None, rec, a, SLOPE, torch.empty_like(Zs[0]),
                              torch.empty((Zs[0].shape[0], H), device="cuda"), ds, torch.zeros_like(a), work[:16])
    assert e.value.code == sar.SAR_ERR_INVALID_ARG
    with pytest.raises(sar.SarError) as e:      # wrong number of source rows: caught by the binding
        sar.sar_gat_fwd_all(b, [Zs[0][:-1], Zs[1]], s, None, a, SLOPE, out, L)
    assert e.value.code == sar.SAR_ERR_INVALID_ARG
    mis = torch.empty(n * H * D + 1, device="cuda")[1:].reshape(n, H, D)      # 4-byte aligned only
    with pytest.raises(sar.SarError) as e:
        sar.sar_gat_fwd_all(b, Zs, s, None, a, SLOPE, mis, L)
    assert e.value.code == sar.SAR_ERR_INVALID_ARG and "aligned" in str(e.value)
    with pytest.raises(sar.SarError) as e:      # neither tq nor a_l
        sar.sar_gat_fwd_all(b, Zs, s, None, None, SLOPE, out, L)
    assert e.value.code == sar.SAR_ERR_INVALID_ARG
    b.close()
    with pytest.raises(sar.SarError):
        b.handle


@pytest.mark.parametrize("dtype,H,D", [(torch.float32, 4, 64), (torch.bfloat16, 8, 32)])
@pytest.mark.parametrize("batched", [False, True])
def test_gat_backward_sources_without_edges(dtype, H, D, batched):
    """Most sources have no edge in their block (a sparse block of a many-way split): their rows of
    dZ_q and dt_q must come back as zeros (the buffers start as NaN), the others as usual."""
    b, want_b, deg, Zdst, Zs, a_l, a_r, G = gat_case(21, 6000, 3000, 3, 1, H, D, dtype, simple=False)
    empty = [np.diff(w.t_indptr) == 0 for w in want_b]
    assert all(e.mean() > 0.5 for e in empty)
    wf = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    wb = orc.gat_bwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE, wf)
    fw = gu.gat_fwd_all(b, Zdst, Zs, a_l, a_r, SLOPE)
    g = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, fw, batched, fly=True)
    for q in range(b.P):
        assert torch.all(g.dZs[q][torch.from_numpy(empty[q]).cuda()] == 0)
        assert torch.all(g.dts[q][torch.from_numpy(empty[q]).cuda()] == 0)
        assert rel_err(f64(g.dZs[q]), wb.dZs[q]) < TOL[dtype], q
        assert rel_err(f64(g.dts[q]), wb.dt[q]) < TOL[dtype], q
    assert rel_err(f64(g.da_l), wb.da_l) < TOL[dtype]
    b.close()


DEGENERATE = {
    "no edges": lambda rng, N, part: ([], [], part, 3, 1),
    "empty destination partition": lambda rng, N, part: (rng.integers(0, N, 200), rng.integers(0, N, 200),
                                                         np.where(part == 1, 0, part), 3, 1),
    "empty source partition": lambda rng, N, part: (rng.integers(0, N, 200), rng.integers(0, N, 200),
                                                    np.where(part == 1, 0, part), 3, 0),
    "single node with a self loop": lambda rng, N, part: ([0], [0], [0], 1, 0),
    "single node without an edge": lambda rng, N, part: ([], [], [0], 1, 0),
    "all edges into one destination": lambda rng, N, part: (rng.integers(0, N, 3000), np.full(3000, 7),
                                                            np.zeros(N, np.int32), 1, 0),
    "all edges out of one source": lambda rng, N, part: (np.full(3000, 7), rng.integers(0, N, 3000),
                                                         np.zeros(N, np.int32), 1, 0),
}


@pytest.mark.parametrize("case", sorted(DEGENERATE))
def test_degenerate_inputs(case):
    """The degenerate cases the method has: nothing to aggregate, nobody to aggregate for, nobody to
    aggregate from, one node, one row that holds every edge.  Tensors without elements are passed
    as they are (null pointers); every call succeeds and agrees with the oracle."""
    rng = np.random.default_rng(3)
    N, H, D = 50, 4, 64
    F = H * D
    part = rng.integers(0, 3, N)
    part[:3] = [0, 1, 2]
    src, dst, part, P, p = DEGENERATE[case](rng, N, part)
    src, dst, part = np.asarray(src, np.int64), np.asarray(dst, np.int64), np.asarray(part, np.int32)
    want_b, deg = orc.build_blocks(src, dst, part, P, p)
    b = gu.build_blocks(src, dst, part, P, p)
    assert b.n_dst == want_b[0].n_dst
    for q in range(P):
        v = gu.view_arrays(b, q)
        assert v["nnz"] == want_b[q].nnz and v["n_src"] == want_b[q].n_src
    Zs = [feats(rng, w.n_src, F, torch.float32).cuda().reshape(-1, H, D) for w in want_b]
    Zdst = feats(rng, b.n_dst, F, torch.float32).cuda().reshape(-1, H, D)
    a_l = torch.from_numpy(rng.uniform(-0.3, 0.3, (H, D)).astype(np.float32)).cuda()
    a_r = torch.from_numpy(rng.uniform(-0.3, 0.3, (H, D)).astype(np.float32)).cuda()
    G = feats(rng, b.n_dst, F, torch.float32).cuda().reshape(-1, H, D)
    Z2, G2 = [z.reshape(-1, F) for z in Zs], G.reshape(-1, F)
    close = lambda got, want: np.allclose(f64(got), want, rtol=0, atol=1e-4 * max(1.0, np.abs(want).max(initial=0)))

    want = orc.spmm(want_b, [f64(z) for z in Z2], True)
    assert close(gu.spmm_all(b, Z2, True), want) and close(gu.spmm_stream(b, Z2, True), want)
    want_d = orc.spmm_bwd(want_b, f64(G2), True)
    d_all = [torch.full_like(z, float("nan")) for z in Z2]
    sar.sar_spmm_bwd_all(b, G2, True, d_all)
    for q in range(P):
        d_blk = torch.full_like(Z2[q], float("nan"))
        sar.sar_spmm_bwd_block(b, q, G2, True, d_blk)
        assert close(d_all[q], want_d[q]) and close(d_blk, want_d[q])

    wf = orc.gat_fwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(a_l), f64(a_r), SLOPE)
    wb = orc.gat_bwd(want_b, f64(Zdst), [f64(z) for z in Zs], f64(G), f64(a_l), f64(a_r), SLOPE, wf)
    for batched in (False, True):
        fw = (gu.gat_fwd_all if batched else gu.gat_fwd_stream)(b, Zdst, Zs, a_l, a_r, SLOPE, fly=True)
        assert close(fw.out, wf.out)
        g = gu.gat_bwd(b, Zdst, Zs, G, a_l, a_r, SLOPE, fw, batched, fly=True)
        for q in range(P):
            assert close(g.dZs[q], wb.dZs[q]) and close(g.dts[q], wb.dt[q])
        assert close(g.dZdst, wb.dZdst) and close(g.ds, wb.ds)
        assert close(g.da_l, wb.da_l) and close(g.da_r, wb.da_r)
    b.close()
