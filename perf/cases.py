"""What a user of the library has it do, as cases that can be timed and compared.

A case is one pass of one worker: a training step or the forward pass of one attention layer (all
blocks resident, or the blocks taken one at a time), a training step of one GraphSage layer, or the
construction of a handle.  `listed()` holds the sizes of this repository's five configurations and of
its head sweep beside smaller, odd and partial ones; `draw()` spreads over the ranges between them.
"""
from __future__ import annotations

import math

import torch

from paper_2111_06483_amd import sar, synth

SLOPE = 0.2
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}

# Layer shapes (heads, head width): the configurations', the head sweep's, the 128-wide attention layer
# of the paper, and those of the parity tests whose heads do not fill a wavefront evenly.
GAT_SHAPES = [(4, 64), (8, 32), (4, 32), (4, 16), (2, 100), (4, 100), (1, 128), (2, 128), (8, 8), (3, 64), (5, 40),
              (2, 50), (1, 47), (3, 12)]
SAGE_WIDTHS = [256, 128, 64, 200, 47, 130, 512]
IN_DIMS = [64, 100, 128, 256]


def listed():
    def case(name, call, graph, N, P, deg, gamma, f_in, H, D, dtype, relu=False, keep=1.0, ship_t=False, compact=True,
             idx64=True):
        return {"name": name, "call": call, "graph": graph, "N": N, "P": P, "deg": deg, "gamma": gamma, "f_in": f_in,
                "H": H, "D": D, "dtype": dtype, "relu": relu, "keep": keep, "ship_t": ship_t, "compact": compact,
                "idx64": idx64}

    return [
        # configuration 1, the smallest layer: a training step whose kernels are short
        case("gat_tiny", "gat", "powerlaw", 4096, 1, 16, 2.1, 64, 4, 16, "f32"),
        # configuration 3, the headline: one worker of eight on the products-sized graph
        case("gat_products", "gat", "powerlaw", 2_450_000, 8, 50, 2.1, 100, 4, 64, "f32"),
        # configuration 4 at half the nodes (three such states fit the card): bf16 rows, most sources
        # with one or two edges in their block
        case("gat_papers_half", "gat", "powerlaw", 55_500_000, 16, 29, 2.2, 128, 8, 32, "bf16"),
        # configuration 5: every row long, no hubs
        case("gat_dense", "gat", "uniform", 200_000, 4, 500, 0.0, 256, 8, 32, "f32"),
        # the head sweep's middle point: the whole graph as one block, rows of 400 values
        case("gat_heads", "gat", "powerlaw", 2_450_000, 1, 50, 2.1, 400, 4, 100, "f32"),
        # the last layer of a network: one head as wide as the classes, an odd width; odd sizes
        case("gat_output", "gat", "powerlaw", 600_011, 4, 50, 2.1, 256, 1, 47, "f32"),
        # a hidden layer restricted to a tenth of the destinations (message flow graph), ReLU, bf16 rows
        case("gat_partial", "gat", "powerlaw", 2_450_000, 8, 50, 2.1, 256, 4, 64, "bf16", relu=True, keep=0.1),
        # the streaming form of the algorithm: one block at a time, the state carried between them, errors of
        # full height; the paper's 128-wide attention layer
        case("gat_blocks", "gat_blocks", "powerlaw", 1_200_000, 16, 29, 2.1, 128, 4, 32, "f32", relu=True, compact=False),
        # inference: the forward pass alone, bf16 rows whose score halves came with them
        case("gat_infer", "gat_fwd", "powerlaw", 5_000_000, 16, 29, 2.2, 128, 8, 32, "bf16", relu=True, ship_t=True),
        # configuration 2: a GraphSage layer with residual and ReLU
        case("sage_products", "sage", "powerlaw", 2_450_000, 8, 50, 2.1, 256, 1, 256, "f32", relu=True),
        # the last GraphSage layer: bf16 rows of 94 bytes
        case("sage_output", "sage", "powerlaw", 1_000_003, 8, 50, 2.1, 256, 1, 47, "bf16"),
        # construction of configuration 3's handle from its edge list
        case("build_products", "build", "powerlaw", 2_450_000, 8, 50, 2.1, 0, 1, 1, "f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["gat"] * 5 + ["gat_fwd", "gat_blocks", "sage", "sage", "build"])
    graph = "uniform" if rng.random() < 0.2 else "powerlaw"
    dtype = rng.choice(["f32", "bf16"])
    H, D = rng.choice(GAT_SHAPES)
    if call == "sage":
        H, D = 1, rng.choice(SAGE_WIDTHS)
    elif call == "build":
        H, D = 1, 1
    # one draw in four has an input width off the usual ones
    f_in = rng.randint(16, 300) if rng.random() < 0.25 else rng.choice(IN_DIMS)
    P = rng.randint(1, 8 if call == "build" else 16)
    N = _log_int(rng, 1_000, 2_500_000)
    deg = _log_int(rng, 4, 100)
    if graph == "uniform":
        deg = _log_int(rng, 4, max(4, min(500, N // 8)))
    # no more gathered bytes and edges than the listed cases of the same data have
    row = H * D * (4 if dtype == "f32" else 2)
    most = min(30_000_000, 30_000_000_000 // row) if call != "build" else 30_000_000
    deg = max(1, min(deg, most * P // N))
    return {"call": call, "graph": graph, "N": N, "P": P, "deg": deg, "gamma": rng.choice([2.1, 2.2]), "f_in": f_in,
            "H": H, "D": D, "dtype": dtype, "relu": rng.random() < 0.5,
            "keep": rng.choice([1.0, 1.0, 0.5, 0.1]) if call in ("gat", "build") else 1.0,
            "ship_t": call in ("gat_fwd", "gat_blocks") and rng.random() < 0.5,
            "compact": rng.random() < 0.75, "idx64": rng.random() < 0.5}


# ------------------------------------------------------------------ what a program holds before the call

class State:
    pass


def _powerlaw_share(case, part):
    """In-edges of worker 0 as `synth.chung_lu_worker_share` draws them, from weights summed as whole numbers:
    a floating prefix sum differs in its last bits from run to run, and with it an edge in many millions."""
    N = case["N"]
    w = (synth.chung_lu_weights(N, case["deg"], case["gamma"], "cuda") * (1 << 20)).to(torch.int64)
    members = torch.nonzero(part == 0).flatten()
    every, own = torch.cumsum(w, 0), torch.cumsum(w[members], 0)
    total_every, total_own, keys = int(every[-1]), int(own[-1]), []
    E, chunk = case["deg"] * members.numel(), 1 << 25
    for lo in range(0, E, chunk):
        ctr = torch.arange(lo, min(E, lo + chunk), device="cuda")
        d = torch.searchsorted(own, (synth.uniform01(0, 12, ctr) * total_own).to(torch.int64), right=True)
        s = torch.searchsorted(every, (synth.uniform01(0, 13, ctr) * total_every).to(torch.int64), right=True)
        keys.append(members[d] * N + s)
    key = torch.unique(torch.cat(keys))
    return key % N, key // N


def _graph(case, seed):
    """Edge list, partition and kept nodes.  Sizes follow from the case alone: its graph and partition are
    drawn once, and the seed then renames the nodes inside windows of 1024 consecutive ids, so that every
    seed has other ids, local ids and index arrays, in blocks of the same sizes.  (Windows, because a
    node's weight falls with its id and ranks near each other have similar weights.)"""
    N, P = case["N"], case["P"]
    part = synth.random_partition(N, P, 1, "cuda")
    if case["graph"] == "powerlaw":
        src, dst = _powerlaw_share(case, part)
    else:
        src, dst = synth.erdos_renyi_worker_share(N, case["deg"], part, 0, 0)
    ids = torch.arange(N, device="cuda")
    keep = synth.uniform01(9, 0, ids) < case["keep"]
    old = torch.argsort(((ids >> 10) << 32) | (synth.hash_counter(seed, 3, ids) & 0xFFFFFFFF))
    new = torch.empty_like(ids)
    new[old] = ids
    key = torch.sort(new[dst] * N + new[src])[0]
    dst, src = key // N, key % N
    part, keep = part[old].contiguous(), keep[old]
    if not case["idx64"]:
        src, dst = src.to(torch.int32), dst.to(torch.int32)
    # the destinations a restricted layer is evaluated for, as local ids, ascending
    kept = torch.nonzero(keep[torch.nonzero(part == 0).flatten()]).flatten().to(torch.int32)
    return part, src, dst, kept


def _flags(case):
    return sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED | (sar.SAR_BUILD_COMPACT if case["compact"] else 0)


def prepare(case, seed):
    s = State()
    s.case, s.seed = case, seed
    P, H, D, f_in = case["P"], case["H"], case["D"], case["f_in"]
    F, dt = H * D, DTYPES[case["dtype"]]
    s.H, s.D, s.F, s.P, s.dt, s.f_in = H, D, F, P, dt, f_in
    s.flags, s.act = _flags(case), sar.SAR_ACT_RELU if case["relu"] else sar.SAR_ACT_NONE
    s.part, s.src, s.dst, ids = _graph(case, seed)
    s.blocks = None
    if case["call"] == "build":
        if case["keep"] < 1.0:      # a restricted handle from a full one
            s.full = sar.sar_blocks_build(s.src, s.dst, s.part, P, 0, s.flags)
            s.ids = ids
        return s

    blocks = sar.sar_blocks_build(s.src, s.dst, s.part, P, 0, s.flags)
    s.part = s.src = s.dst = None
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def randn(*shape, dtype=dt):
        return torch.randn(*shape, dtype=dtype, device="cuda", generator=g)

    def empty(*shape, dtype=dt):
        return torch.empty(*shape, dtype=dtype, device="cuda")

    f32 = torch.float32
    s.n_own = blocks.n_src(0)
    s.X = randn(s.n_own, f_in)
    s.Xd = s.X
    s.partial = case["keep"] < 1.0
    if s.partial:
        s.full = blocks
        blocks = sar.sar_blocks_subset(s.full, ids, s.flags)
        s.Xd = s.X[ids.long()].contiguous()
    s.blocks, s.n = blocks, blocks.n_dst
    s.views = [blocks.view(q) for q in range(P)]
    s.W, s.a_l, s.a_r = synth.gat_params(seed, f_in, H, D, device="cuda")
    # the other partitions' rows as fetched: they have the distribution of rows x W with N(0,1) inputs
    spread = math.sqrt(2.0 * f_in / (f_in + F))
    s.Zs = [None] + [randn(blocks.n_src(q), H, D).mul_(spread) for q in range(1, P)]
    s.Zp = empty(s.n_own, H, D)
    s.out = empty(s.n, H, D)
    s.L = empty(s.n, H, dtype=f32)
    s.s = empty(s.n, H, dtype=f32)
    s.tp = empty(s.n, H, dtype=f32)
    s.tq = None
    if case["ship_t"]:
        s.tq = [empty(blocks.n_src(q), H, dtype=f32) for q in range(P)]
        for q in range(1, P):
            sar.sar_gat_scores(s.Zs[q], s.a_l, s.tq[q])
        s.tp = s.tq[0]
    if case["call"] == "gat_fwd":
        return s

    s.G = randn(s.n, H, D)
    s.dZs = [empty(blocks.n_err_rows(q), H, D) for q in range(P)]
    s.dX = empty(s.n, f_in)
    s.lwork = empty(max(1, sar.sar_linear_workspace_bytes(s.n_own, f_in, F) // 4), dtype=f32)
    s.rank = s.views[0].t_rank if case["compact"] else None
    s.rows = None
    if case["call"] == "sage":
        s.W_res = synth.xavier_uniform(seed, 3, (f_in, F), f_in, F, "cuda")
        s.R, s.G2 = empty(s.n, F), empty(s.n, F)
        s.grads = empty(2 * f_in * F, dtype=f32)
        s.dW, s.dW_res = s.grads[: f_in * F].view(f_in, F), s.grads[f_in * F:].view(f_in, F)
        s.dX_res = empty(s.n, f_in)
        return s

    s.Zd = empty(s.n, H, D) if s.partial else s.Zp
    s.rec, s.ds = empty(s.n, H, 4, dtype=f32), empty(s.n, H, dtype=f32)
    s.Gact = empty(s.n, H, D) if case["relu"] else None
    s.grads = empty(2 * F + f_in * F, dtype=f32)
    s.da_l, s.da_r = s.grads[:F].view(H, D), s.grads[F:2 * F].view(H, D)
    s.dW = s.grads[2 * F:].view(f_in, F)
    s.work = empty(sar.sar_gat_workspace_bytes(s.n, max(blocks.n_src(q) for q in range(P)), H, D) // 4, dtype=f32)
    if s.partial:
        s.E_own, s.dX_own = empty(s.n_own, H, D), empty(s.n_own, f_in)
    if case["call"] == "gat_blocks":
        s.m, s.l, s.acc = empty(s.n, H, dtype=f32), empty(s.n, H, dtype=f32), empty(s.n, H, D, dtype=f32)
    return s


# ------------------------------------------------------------------------------------------- one pass

def _bwd_rows(s, E, rank, ds, a_r, H, D, W, dW, dX):
    """dW += X^T E_p, dX = E_p W^T with the rows of E_p formed in the products where the shape allows it,
    else written to scratch that the program keeps."""
    args = (s.Xd, E, rank, ds, a_r, H, D, W, dW, dX, s.n, s.dt, s.lwork)
    try:
        sar.sar_linear_bwd_rows(*args, rows=s.rows)
    except sar.SarError as e:
        if e.code != sar.SAR_ERR_UNSUPPORTED or s.rows is not None:
            raise
        s.rows = torch.empty((s.n, s.F), dtype=s.dt, device="cuda")
        sar.sar_linear_bwd_rows(*args, rows=s.rows)


def _gat_forward(s, blockwise):
    Zd = s.Zp if s.case["call"] == "gat_fwd" else s.Zd
    # Eq. 1 for the worker's own rows, with both score halves
    sar.sar_linear_fwd(s.Xd, s.W, Zd.view(s.n, s.F), s.a_r, s.s, s.a_l, s.tp)
    if Zd is not s.Zp:                       # the local block reads every own row as a source
        sar.sar_linear_fwd(s.X, s.W, s.Zp.view(s.n_own, s.F))
    Zs = [s.Zp] + s.Zs[1:]
    if not blockwise:
        sar.sar_gat_fwd_all(s.blocks, Zs, s.s, s.tq, s.a_l, SLOPE, s.out, s.L, s.act)
        return Zs
    sar.sar_gat_fwd_begin(s.m, s.l, s.acc)
    for q in range(s.P):
        sar.sar_gat_fwd_block(s.blocks, q, Zs[q], s.s, None if s.tq is None else s.tq[q], s.a_l, SLOPE, s.m, s.l, s.acc)
    sar.sar_gat_fwd_end(s.m, s.l, s.acc, s.out, s.L, s.act)
    return Zs


def _gat_step(s, blockwise):
    Zs = _gat_forward(s, blockwise)
    sar.sar_gat_bwd_begin(s.G, s.out, s.s, s.L, s.rec, s.ds, s.act, s.Gact)
    G = s.Gact if s.act else s.G
    s.grads.zero_()
    if blockwise:
        for q in range(s.P):
            sar.sar_gat_bwd_block(s.blocks, q, Zs[q], G, None if s.tq is None else s.tq[q], s.rec, s.a_l, SLOPE,
                                  s.dZs[q], None, s.ds, s.da_l, s.work)
    else:
        sar.sar_gat_bwd_all(s.blocks, Zs, G, s.tq, s.rec, s.a_l, SLOPE, s.dZs, None, s.ds, s.da_l, s.work)
    sar.sar_gat_bwd_end(s.Zd, s.ds, s.a_r, None, None, s.da_r, s.work)           # da_r
    own = s.dZs[0]
    if not s.partial:
        _bwd_rows(s, own.view(-1, s.F), s.rank, s.ds, s.a_r, s.H, s.D, s.W, s.dW, s.dX)
        return {"out": s.out, "L": s.L, "dZ": s.dZs, "ds": s.ds, "da_l": s.da_l, "da_r": s.da_r, "dW": s.dW, "dX": s.dX}
    # destination and source roles of the own rows apart: the listed rows get the score term, all own rows
    # the local block's error
    _bwd_rows(s, None, None, s.ds, s.a_r, s.H, s.D, s.W, s.dW, s.dX)
    if s.rank is not None:
        sar.sar_error_add(own, s.rank, False, s.E_own)
        own = s.E_own
    sar.sar_linear_bwd(s.X, own, s.W, s.dW, s.dX_own, s.lwork)
    return {"out": s.out, "L": s.L, "dZ": s.dZs, "ds": s.ds, "da_l": s.da_l, "da_r": s.da_r, "dW": s.dW, "dX": s.dX,
            "dX_own": s.dX_own}


def _sage_step(s):
    n, F = s.n, s.F
    Zp, h, G = s.Zp.view(n, F), s.out.view(n, F), s.G.view(n, F)
    sar.sar_linear_fwd(s.X, s.W, Zp)
    sar.sar_linear_fwd(s.X, s.W_res, s.R)
    sar.sar_spmm_all(s.blocks, [Zp] + [z.view(-1, F) for z in s.Zs[1:]], True, h, s.R, s.act)
    if s.act:
        sar.sar_act_bwd(h, G, s.act, s.G2)
        G = s.G2
    s.grads.zero_()
    dZs = [e.view(-1, F) for e in s.dZs]
    sar.sar_spmm_bwd_all(s.blocks, G, True, dZs)
    sar.sar_linear_bwd(s.X, G, s.W_res, s.dW_res, s.dX_res, s.lwork)
    _bwd_rows(s, dZs[0], s.rank, None, None, 1, F, s.W, s.dW, s.dX)
    return {"h": h, "dZ": dZs, "dW": s.dW, "dW_res": s.dW_res, "dX": s.dX, "dX_res": s.dX_res}


class _DeviceInts:
    """An index array of a handle, lent to torch without a copy; the tensor made of it keeps the handle."""

    def __init__(self, blocks, ptr, count):
        self.blocks = blocks
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<i4", "data": (ptr, False), "version": 3,
                                         "strides": None}


def _ints(blocks, ptr, count):
    if not count or not ptr:
        return torch.empty(0, dtype=torch.int32, device="cuda")
    return torch.as_tensor(_DeviceInts(blocks, ptr, count), device="cuda")


def _build(s):
    if s.case["keep"] < 1.0:
        b = sar.sar_blocks_subset(s.full, s.ids, s.flags)
    else:
        b = sar.sar_blocks_build(s.src, s.dst, s.part, s.P, 0, s.flags)
    s.blocks = b                             # a program keeps the newest handle
    out = {"deg": sar.sar_blocks_degree(b)}
    for q in range(s.P):
        v = b.view(q)
        out["block%d" % q] = [_ints(b, p, n) for p, n in ((v.indptr, v.n_dst + 1), (v.indices, v.nnz),
                                                          (v.t_indptr, v.n_src + 1), (v.t_indices, v.nnz),
                                                          (v.touched, v.n_t_rows), (v.t_rank, v.n_src + 1))]
    return out


def run(s):
    call = s.case["call"]
    if call == "gat":
        return _gat_step(s, False)
    if call == "gat_blocks":
        return _gat_step(s, True)
    if call == "gat_fwd":
        _gat_forward(s, False)
        return {"Z": s.Zp, "s": s.s, "t": s.tp, "out": s.out, "L": s.L}
    if call == "sage":
        return _sage_step(s)
    return _build(s)


# -------------------------------------------------------------------------- work and agreement of a pass

def _touched(case, E):
    """Expected number of sources with an edge into the worker's destinations.  A source of weight w is
    drawn Poisson(E w / sum w) times; the weights (v + v0)^-b of `synth.chung_lu_weights` are integrated
    here instead of being laid out for every node."""
    N = case["N"]
    if case["graph"] == "uniform":
        return N * (1.0 - math.exp(-E / N))
    b, deg = 1.0 / (case["gamma"] - 1.0), float(case["deg"])

    def total(v0):
        return ((N + v0) ** (1.0 - b) - v0 ** (1.0 - b)) / (1.0 - b)

    lo, hi = 1e-6, float(N)
    for _ in range(60):
        mid = math.sqrt(lo * hi)
        lo, hi = (mid, hi) if deg * N / total(mid) * mid ** -b > math.sqrt(N * deg) else (lo, mid)
    v0 = math.sqrt(lo * hi)
    scale, parts = E / total(v0), 20_000
    step = (math.log(N + v0) - math.log(v0)) / parts
    got = 0.0
    for k in range(parts):                   # midpoints of equal steps of log(v + v0)
        x = math.exp(math.log(v0) + (k + 0.5) * step)
        got += (1.0 - math.exp(-scale * x ** -b)) * x * step
    return got


def work(case):
    """Inputs read once, outputs written once (the handle's index arrays are inputs; tensors that one call
    leaves for the next one are neither); multiply-adds of the products and of the rows along the edges."""
    P, F, H, f_in = case["P"], case["H"] * case["D"], case["H"], case["f_in"]
    fb = 4 if case["dtype"] == "f32" else 2
    n_own = -(-case["N"] // P)
    n = n_own * case["keep"]
    E = n * case["deg"]
    U = _touched(case, E)
    if case["call"] == "build":
        idx = 8 if case["idx64"] else 4
        given = 4 * E + 4 * n * (P + 1) if case["keep"] < 1.0 else 2 * idx * E + 4 * case["N"]
        # CSR, transpose and the index over all blocks; row offsets, touched lists and ranks
        return {"bytes": given + 12 * E + 4 * (P + 2) * n + 8 * case["N"] + 4 * U, "flops": 0}
    rows = U * F * fb
    fetched = rows * (P - 1) / P             # the local block's rows are made in the pass
    index = 4 * E + 4 * n
    edges = 2 * E * F + 2 * U * F
    x = n_own * f_in * fb
    if case["call"] == "gat_fwd":
        shipped = 4 * H * U if case["ship_t"] else 0
        return {"bytes": x + fetched + shipped + index + n * (2 * F * fb + 12 * H), "flops": 2 * n * f_in * F + edges}
    if case["call"] == "sage":
        return {"bytes": 3 * x + fetched + rows + 2 * index + 2 * n * F * fb + 16 * f_in * F,
                "flops": 12 * n * f_in * F + 4 * E * F}
    products = 6 * n * f_in * F
    if case["keep"] < 1.0:
        x, products = x * (2 + 2 * case["keep"]), products + 6 * n_own * f_in * F
    else:
        x = 2 * x
    return {"bytes": x + fetched + rows + 2 * index + n * (2 * F * fb + 8 * H) + 8 * f_in * F,
            "flops": products + edges + 4 * E * F + 2 * U * F}


def tolerance(case):
    """Sums are taken in 32 bits everywhere; bf16 rows are rounded when stored.  The attention gradients are
    looser than their sums: the slope of the LeakyReLU is chosen by the sign of a 32-bit score, and an edge
    whose score is zero within rounding carries one slope or the other (about one edge in 100,000), which
    moves ds of its row by a whole term and the parameters' gradients, whose terms nearly cancel, by some
    1e-4 of their size."""
    if case["call"] == "build":
        return "exact"
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.5}
    if case["call"] in ("gat", "gat_blocks"):
        return {"rel": 5e-4, "max": 0.5}
    return {"rel": 1e-5, "max": 1e-3}
