"""Dense graphs, whose all-blocks passes go by head slices (gat_slices.h): forward with and without barriers, backward, the
heads and widths they take, rows that end inside a batch or have no edge, against the same layer block by block (the
kernels of gat_f256.h and gat_slots.h, which the oracle tests hold; the source score halves are formed in the same order,
so both sides choose the same slopes)."""
import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def layer(n_own, n_other, P, deg, H, D, dtype, seed, compact):
    """Every destination but each 97th has about `deg` sources, uniform over P partitions (the first is the worker's)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    N = n_own + (P - 1) * n_other
    part = torch.cat([torch.zeros(n_own, dtype=torch.int64), 1 + torch.arange((P - 1) * n_other) // max(n_other, 1)])
    keep = torch.arange(n_own, device="cuda") % 97 != 3
    keep[0] = False                                    # the first row of the index and the last one empty
    keep[-1] = False
    counts = (deg + torch.randint(-deg // 4, deg // 4 + 1, (n_own,), generator=g, device="cuda")) * keep
    dst = torch.repeat_interleave(torch.arange(n_own, device="cuda"), counts)
    src = torch.randint(0, N, (int(counts.sum()),), generator=g, device="cuda")
    key = torch.unique(dst * N + src)
    dst, src = key // N, key % N
    flags = sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | (sar.SAR_BUILD_COMPACT if compact else 0)
    b = sar.sar_blocks_build(src, dst, part.to(torch.int32).cuda(), P, 0, flags)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    Zs = [(rnd(b.n_src(q), H, D)).to(dtype) for q in range(P)]
    a_l, a_r = rnd(H, D) / D ** 0.5, rnd(H, D) / D ** 0.5
    return b, Zs, a_l, a_r, rnd(n_own, H, D).to(dtype)


def kernels_of(call):
    """Names of the kernels that a call launches."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in p.events())


def close(got, want, tol):
    got, want = got.double(), want.double()
    assert torch.equal(torch.isfinite(got), torch.isfinite(want))
    ok = torch.isfinite(want)
    scale = float(want[ok].abs().max())
    assert float((got[ok] - want[ok]).abs().max()) <= tol * scale


# (destinations, other sources, partitions, edges a row).  Barriers: a head's table beyond 3 MiB, the whole one from 24 MiB on,
# four sweeps and more of two and five uses, in both passes of the first four (backward: fp32, G from 28 MiB on) and in
# the forward pass of the other four; no barriers: the small tables behind.
SHAPES = [(30_000, 2_000, 2, 90, 8, 32), (30_000, 2_000, 2, 90, 4, 64), (58_000, 3_000, 2, 130, 1, 128),
          (30_000, 1_500, 3, 90, 2, 128), (17_000, 16_000, 2, 75, 2, 100), (16_390, 28_000, 2, 50, 4, 36),
          (33_000, 9_000, 3, 80, 4, 32), (8_200, 8_000, 2, 45, 16, 64), (9_000, 300, 2, 30, 16, 40), (23_000, 500, 2, 9, 8, 32)]


@pytest.mark.parametrize("n_own,n_other,P,deg,H,D", SHAPES)
@pytest.mark.parametrize("dtype,shipped,relu,compact", [(torch.float32, False, False, True), (torch.float32, True, True, False),
                                                        (torch.bfloat16, False, True, True)])
def test_layer(n_own, n_other, P, deg, H, D, dtype, shipped, relu, compact):
    b, Zs, a_l, a_r, G = layer(n_own, n_other, P, deg, H, D, dtype, seed=n_own + H, compact=compact)
    act = sar.SAR_ACT_RELU if relu else sar.SAR_ACT_NONE
    n, f32 = b.n_dst, torch.float32
    tq = None
    if shipped:
        tq = [torch.empty(b.n_src(q), H, device="cuda") for q in range(P)]
        for q in range(P):
            sar.sar_gat_scores(Zs[q], a_l, tq[q])
    s = torch.empty(n, H, device="cuda")
    sar.sar_gat_scores(Zs[0], a_r, s)
    out, L = torch.full((n, H, D), 7.0, device="cuda", dtype=dtype), torch.full((n, H), 7.0, device="cuda")
    sar.sar_gat_fwd_all(b, Zs, s, tq, a_l, 0.2, out, L, act)
    m, l, acc = torch.empty(n, H, device="cuda"), torch.empty(n, H, device="cuda"), torch.empty(n, H, D, device="cuda")
    sar.sar_gat_fwd_begin(m, l, acc)
    for q in range(P):
        sar.sar_gat_fwd_block(b, q, Zs[q], s, None if tq is None else tq[q], a_l, 0.2, m, l, acc)
    out2, L2 = torch.empty_like(out), torch.empty_like(L)
    sar.sar_gat_fwd_end(m, l, acc, out2, L2, act)
    # (fp32: sums of a hundred terms in another order; bf16: one rounding of the stored row)
    close(out, out2, 2e-6 if dtype == f32 else 2.0 ** -8)
    close(L, L2, 2e-6)
    assert (out.reshape(n, -1)[0] == 0).all() and L[0].isneginf().all()

    rec, ds0 = torch.empty(n, H, 4, device="cuda"), torch.empty(n, H, device="cuda")
    Ga = torch.empty_like(G) if relu else None
    sar.sar_gat_bwd_begin(G, out, s, L, rec, ds0, act, Ga)
    Gb = Ga if relu else G
    full = sar.sar_gat_workspace_bytes(n, max(b.n_src(q) for q in range(P)), H, D)
    least = 4 * 2048 * 256 * 4
    assert full > least
    res = []
    for size in (full, least):            # with the least scratch the pass takes its other way
        dZ = [torch.full((b.n_err_rows(q), H, D), float("nan"), device="cuda", dtype=dtype) for q in range(P)]
        dt = [torch.full((b.n_err_rows(q), H), float("nan"), device="cuda") for q in range(P)]
        ds, da = torch.zeros(n, H, device="cuda"), torch.zeros(H, D, device="cuda")
        work = torch.full((size // 4,), float("nan"), device="cuda")
        sar.sar_gat_bwd_all(b, Zs, Gb, tq, rec, a_l, 0.2, dZ, dt, ds, da, work)
        res.append((dZ, dt, ds, da))
    for x, y in zip(res[0][0], res[1][0]):
        close(x, y, 2e-6 if dtype == f32 else 2.0 ** -8)
    for x, y in zip(res[0][1], res[1][1]):
        close(x, y, 1e-5)
    close(res[0][2], res[1][2], 1e-5)
    close(res[0][3], res[1][3], 1e-5)


@pytest.mark.parametrize("n_own,n_other,P,deg,H,D", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_which_kernels_run(n_own, n_other, P, deg, H, D, dtype):
    """The shapes above reach what they are there for: forward slices with barriers (tables beyond 3 MiB) or without, and
    backward slices where scratch is given for them."""
    b, Zs, a_l, a_r, G = layer(n_own, n_other, P, deg, H, D, dtype, seed=1, compact=True)
    n, f32 = b.n_dst, dtype == torch.float32
    s = torch.zeros(n, H, device="cuda")
    out, L = torch.empty(n, H, D, device="cuda", dtype=dtype), torch.empty(n, H, device="cuda")
    index = SHAPES.index((n_own, n_other, P, deg, H, D))
    tq = [torch.zeros(b.n_src(q), H, device="cuda") for q in range(P)]
    for given in (None, tq):
        names = kernels_of(lambda: sar.sar_gat_fwd_all(b, Zs, s, given, a_l, 0.2, out, L, sar.SAR_ACT_NONE))
        if f32:
            assert "k_gat_fwd_slices" in names and ("true>" in names) == (index < 8)
        elif D < 64 or index >= 8:
            assert "k_gat_fwd_slices" not in names
    rec, ds = torch.empty(n, H, 4, device="cuda"), torch.empty(n, H, device="cuda")
    sar.sar_gat_bwd_begin(G, out, s, L, rec, ds)
    dZ = [torch.empty(b.n_err_rows(q), H, D, device="cuda", dtype=dtype) for q in range(P)]
    full = sar.sar_gat_workspace_bytes(n, max(b.n_src(q) for q in range(P)), H, D)
    for size in (full, 4 * 2048 * 256 * 4):
        work, da = torch.empty(size // 4, device="cuda"), torch.zeros(H, D, device="cuda")
        names = kernels_of(lambda: sar.sar_gat_bwd_all(b, Zs, G, None, rec, a_l, 0.2, dZ, None, ds, da, work))
        assert ("k_gat_bwd_slices" in names) == (f32 and index < 4 and size == full)


@pytest.mark.parametrize("H,D,n_own", [(8, 32, 30_000), (4, 64, 30_000), (2, 64, 58_000), (2, 128, 30_000)])
@pytest.mark.parametrize("flags", [0, sar.SAR_BUILD_COMPACT, sar.SAR_BUILD_COMPACT | sar.SAR_BUILD_SINGLES])
@pytest.mark.parametrize("hub", [False, True])
def test_sources_of_all_kinds(H, D, n_own, flags, hub):
    """Sources of 90 or 140 edges by slices beside sources of 0, 1 and 2 to 7 edges by the other kernels of the same call, ds
    summed in copies where one destination is cited by all: against the call whose scratch has no room for slices."""
    g = torch.Generator(device="cuda").manual_seed(H * D + n_own)
    kinds = [(n_own, 90 if n_own < 50_000 else 140)] + [(3000, k) for k in (0, 1, 1, 2, 3, 5, 7, 8, 9)]
    counts = torch.cat([torch.full((n,), k, device="cuda") for n, k in kinds])
    N = counts.numel()
    src = torch.repeat_interleave(torch.arange(N, device="cuda"), counts)
    dst = torch.randint(0, n_own, (src.numel(),), generator=g, device="cuda")
    if hub:
        dst[torch.cumsum(counts, 0)[counts > 1] - 1] = 17
    key = torch.unique(dst * N + src)
    part = torch.cat([torch.zeros(n_own, dtype=torch.int32), 1 + torch.arange(N - n_own, dtype=torch.int32) % 2])
    b = sar.sar_blocks_build(key % N, key // N, part.cuda(), 3, 0, sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | flags)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    Zs = [rnd(b.n_src(q), H, D) for q in range(3)]
    a_l, a_r, G, n = rnd(H, D) / D ** 0.5, rnd(H, D) / D ** 0.5, rnd(n_own, H, D), n_own
    s, out, L = torch.empty(n, H, device="cuda"), torch.empty(n, H, D, device="cuda"), torch.empty(n, H, device="cuda")
    sar.sar_gat_scores(Zs[0], a_r, s)
    sar.sar_gat_fwd_all(b, Zs, s, None, a_l, 0.2, out, L, sar.SAR_ACT_NONE)
    rec, ds0 = torch.empty(n, H, 4, device="cuda"), torch.empty(n, H, device="cuda")
    sar.sar_gat_bwd_begin(G, out, s, L, rec, ds0)
    full, res = sar.sar_gat_workspace_bytes(n, max(b.n_src(q) for q in range(3)), H, D), []
    for size in (full, full - n * H * 20):
        dZ = [torch.full((b.n_err_rows(q), H, D), float("nan"), device="cuda") for q in range(3)]
        dt = [torch.full((b.n_err_rows(q), H), float("nan"), device="cuda") for q in range(3)]
        ds, da = torch.zeros(n, H, device="cuda"), torch.zeros(H, D, device="cuda")
        work = torch.full((size // 4,), float("nan"), device="cuda")
        names = kernels_of(lambda: sar.sar_gat_bwd_all(b, Zs, G, None, rec, a_l, 0.2, dZ, dt, ds, da, work))
        assert ("k_gat_bwd_slices" in names) == (size == full) and ("k_ds_sum" in names) == hub
        res.append((dZ, dt, ds, da))
    for x, y in zip(res[0][0] + res[0][1], res[1][0] + res[1][1]):
        close(x, y, 1e-5)
    # (17 of the hub's row: the sum of 40 thousand terms in another order)
    close(res[0][2], res[1][2], 1e-5 if not hub else 40_000 ** 0.5 * 2.0 ** -24)
    close(res[0][3], res[1][3], 1e-5)


@pytest.mark.parametrize("n_own,n_other,P,deg,H,D", [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[4], SHAPES[6], SHAPES[9]])
def test_infinities_stay_with_their_edges(n_own, n_other, P, deg, H, D):
    """An infinity in the last row that a destination (backward: a source) gathers, with longer rows beside it: the result
    it belongs to is infinite and no result is NaN."""
    b, Zs, a_l, a_r, G = layer(n_own, n_other, P, deg, H, D, torch.float32, seed=D, compact=False)
    n, inf = b.n_dst, float("inf")
    edges = []          # (destination, local source) by block
    for q in range(P):
        v = gu.view_arrays(b, q)
        ip, ix = (torch.as_tensor(v[k]).long().cuda() for k in ("indptr", "indices"))
        edges.append((torch.repeat_interleave(torch.arange(n, device="cuda"), ip[1:] - ip[:-1]), ix))
    a_l, Zs, G = a_l.abs() + 0.01, [z.abs() + 0.01 for z in Zs], G.abs() + 0.01
    tq = [torch.empty(b.n_src(q), H, device="cuda") for q in range(P)]
    for q in range(P):
        sar.sar_gat_scores(Zs[q], a_l, tq[q])
    s = torch.zeros(n, H, device="cuda")
    out, L = torch.empty(n, H, D, device="cuda"), torch.empty(n, H, device="cuda")
    sar.sar_gat_fwd_all(b, Zs, s, tq, a_l, 0.2, out, L, sar.SAR_ACT_NONE)
    rec, ds = torch.empty(n, H, 4, device="cuda"), torch.empty(n, H, device="cuda")
    sar.sar_gat_bwd_begin(G, out, s, L, rec, ds)

    dst, src = edges[P - 1]
    last = int(src.max())
    Zi = [z.clone() for z in Zs]
    Zi[P - 1][last, 0, D - 1] = inf
    out2 = torch.empty_like(out)
    sar.sar_gat_fwd_all(b, Zi, s, tq, a_l, 0.2, out2, torch.empty_like(L), sar.SAR_ACT_NONE)
    want = torch.isinf(out)
    want[dst[src == last], 0, D - 1] = True
    assert bool(want.any()) and torch.equal(out2 == inf, want) and not torch.isnan(out2).any()

    if (n_own, n_other, P, deg, H, D) not in SHAPES[:4]:       # (the backward pass by other kernels)
        return
    i = max(int(d.max()) for d, _ in edges)
    Gi = G.clone()
    Gi[i, 0, 0] = inf
    dZ = [torch.zeros(b.n_src(q), H, D, device="cuda") for q in range(P)]
    work = torch.empty(sar.sar_gat_workspace_bytes(n, max(b.n_src(q) for q in range(P)), H, D) // 4, device="cuda")
    sar.sar_gat_bwd_all(b, Zs, Gi, tq, rec, a_l, 0.2, dZ, None, ds, torch.zeros(H, D, device="cuda"), work)
    for q in range(P):
        want = torch.zeros(b.n_src(q), H, dtype=torch.bool, device="cuda")
        want[edges[q][1][edges[q][0] == i], 0] = True
        assert torch.equal((dZ[q] == inf).all(-1), want) and not torch.isnan(dZ[q]).any()
