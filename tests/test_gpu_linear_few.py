"""The transform of few rows against the kernels that many rows take: a row's results do not depend on how many rows
a call has, so the first rows of a large call are the reference, bit for bit."""
import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MANY = 70_000       # beyond the lines of every width below

# tiles of one column to several, contractions that end inside a piece, a chunk, a ring of chunks; heads of any width
SHAPES = [(64, 4, 16), (36, 1, 33), (100, 4, 64), (128, 3, 20), (256, 8, 32), (255, 1, 47), (72, 2, 50), (300, 5, 12), (21, 1, 130)]


def layer(K, H, D, dtype):
    g = torch.Generator(device="cuda").manual_seed(K * 1000 + H * D)
    draw = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
    return (draw(MANY, K).to(dtype), draw(MANY, H * D).to(dtype), draw(K, H * D) / K ** 0.5, draw(H, D), draw(H, D),
            draw(MANY, H))


@pytest.mark.parametrize("K,H,D", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("scores", [0, 1, 2])
def test_forward(K, H, D, dtype, scores):
    X, _, W, a, b, _ = layer(K, H, D, dtype)

    def run(n):
        Z = torch.empty(n, H * D, dtype=dtype, device="cuda")
        s, t = torch.empty(n, H, device="cuda"), torch.empty(n, H, device="cuda")
        second = (b, t) if scores == 2 else (None, None)
        sar.sar_linear_fwd(X[:n], W, Z, *((a, s) if scores else (None, None)), *second)
        return [Z, s, t][: 1 + scores]

    assert "k_few" not in gu.kernels_of(lambda: run(MANY)) and "k_few" in gu.kernels_of(lambda: run(1000))
    want = run(MANY)
    for n in (1, 32, 33, 127, 1000):
        for got, many in zip(run(n), want):
            assert torch.equal(got, many[:n])


@pytest.mark.parametrize("K,H,D", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("formed", [False, True])
def test_backward(K, H, D, dtype, formed):
    X, E, W, a, _, ds = layer(K, H, D, dtype)
    F = H * D

    def run(n):
        work = torch.empty(max(1, sar.sar_linear_workspace_bytes(n, K, F) // 4), device="cuda")
        dW, dX = torch.ones(K, F, device="cuda"), torch.empty(n, K, dtype=dtype, device="cuda")
        if not formed:
            sar.sar_linear_bwd(X[:n], E[:n], W, dW, dX, work)
            return dW, dX, E[:n].double()
        # every third row has no stored part
        has = torch.arange(n, device="cuda") % 3 != 1
        rank = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
        rank[1:] = torch.cumsum(has, 0)
        stored = E[:n][has].contiguous()
        sar.sar_linear_bwd_rows(X[:n], stored, rank.data_ptr(), ds[:n].contiguous(), a, H, D, W, dW, dX, n, dtype, work)
        rows = torch.where(has[:, None], E[:n], 0).double() + (ds[:n, :, None].double() * a.double()).reshape(n, F)
        return dW, dX, rows.to(dtype).double()

    try:
        _, want, _ = run(MANY)
    except sar.SarError as e:
        assert formed and e.code == sar.SAR_ERR_UNSUPPORTED      # (the same shapes are refused for any number of rows)
        with pytest.raises(sar.SarError):
            run(100)
        return
    assert "k_few" not in gu.kernels_of(lambda: run(MANY)) and "k_few" in gu.kernels_of(lambda: run(1500))
    # (n, groups of 32 rows: one, one for each wavefront, one slab, several)
    for n in (1, 2, 31, 128, 129, 640, 641, 1500):
        dW, dX, rows = run(n)
        assert torch.equal(dX, want[:n])
        # (F products, as above; bf16: the stored result's rounding, 2^-8 of a value at most, and those of the formed rows)
        back = rows @ W.double().T
        off = max(2.0, F ** 0.5) * 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8 * (1.1 if formed else 1.0)
        assert float((dX.double() - back).norm() / back.norm()) < off
        exact = 1.0 + X[:n].double().T @ rows
        # a sum of n products: n^1/2 roundings of the running sum, below 2^-24 of its scale each, and (bf16) those of the
        # formed rows, which 64 bits round to the other neighbour where fp32's multiply-add is within its rounding of a tie
        tol = max(2.0, n ** 0.5) * 2.0 ** -24 + (2.0 ** -9 * 0.1 if formed and dtype == torch.bfloat16 else 0.0)
        assert float((dW.double() - exact).norm() / exact.norm()) < tol


@pytest.mark.parametrize("n", [1, 100, MANY])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_neither_product_wanted(n, dtype):
    """dW and dX may each be left out, so may both, for any number of rows; `rows` is written all the same."""
    X, E, W, a, _, ds = layer(64, 4, 16, dtype)
    sar.sar_linear_bwd(X[:n], E[:n], W, None, None, None)
    sar.sar_linear_bwd_rows(X[:n], E[:n], None, ds[:n], a, 4, 16, W, None, None, n, dtype, None)
    rows = torch.full((n, 64), float("nan"), dtype=dtype, device="cuda")
    sar.sar_linear_bwd_rows(X[:n], E[:n], None, None, None, 4, 16, W, None, None, n, dtype, None, rows=rows)
    assert torch.equal(rows, E[:n])


def test_result_over_an_operand():
    """Z over X and dX over dZ go the other kernels' way: a tile's rows are read again after others are stored."""
    X = torch.randn(500, 64, device="cuda")
    W = torch.randn(64, 64, device="cuda") / 8
    Z, dX = torch.empty_like(X), torch.empty_like(X)
    sar.sar_linear_fwd(X, W, Z)
    sar.sar_linear_bwd(None, X, W, None, dX, None)
    A, B = X.clone(), X.clone()
    sar.sar_linear_fwd(A, W, A)
    sar.sar_linear_bwd(None, B, W, None, B, None)
    assert torch.equal(A, Z)
    want = X.double() @ W.double().T
    assert float((B.double() - want).norm() / want.norm()) < 8 * 2.0 ** -24
    assert float((dX.double() - want).norm() / want.norm()) < 8 * 2.0 ** -24


@pytest.mark.parametrize("n,K,F,dtype", [(8192, 256, 512, torch.bfloat16), (16384, 128, 400, torch.bfloat16), (2560, 512, 384, torch.float32),
                                         (20480, 64, 256, torch.float32), (1500, 256, 256, torch.bfloat16), (8192, 128, 2048, torch.bfloat16),
                                         (8192, 256, 400, torch.bfloat16), (2048, 512, 1024, torch.float32), (2560, 512, 256, torch.float32)])
@pytest.mark.parametrize("alone", [True, False])
def test_weight_gradients_of_long_slabs(n, K, F, dtype, alone):
    """Many columns leave few slabs, of hundreds of rows for a wavefront.  Normal operands: a result is of size n^1/2, and so is
    a partial sum of m rows of size m^1/2; eight sums of 32 rows, up to eight of those and four wavefronts' and eight slabs'
    sums are some 17 n of squares in all, each rounded by 0.42 of 2^-24 in the mean: 1.7 2^-24 of the result (measured: 1.7)."""
    g = torch.Generator(device="cuda").manual_seed(n + K)
    X, dZ = (torch.randn(n, w, device="cuda", generator=g).to(dtype) for w in (K, F))
    W = torch.randn(K, F, device="cuda", generator=g)
    work = torch.empty(sar.sar_linear_workspace_bytes(n, K, F) // 4, device="cuda")
    dW, dX = torch.zeros(K, F, device="cuda"), None if alone else torch.empty_like(X)
    sar.sar_linear_bwd(X, dZ, None if alone else W, dW, dX, work)
    want = X.double().T @ dZ.double()
    assert float((dW.double() - want).norm() / want.norm()) < 2.0 * 2.0 ** -24


@pytest.mark.parametrize("stored", [0, 40])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_results_do_not_depend_on_where_operands_lie(stored, dtype):
    """dX right behind the few stored rows of a compact E, or behind a_r where no row is stored: the same bits as far off."""
    n, K, H, D = 1500, 64, 4, 16
    F = H * D
    X, E, W, a, _, ds = layer(K, H, D, dtype)
    rank = torch.arange(n + 1, dtype=torch.int32, device="cuda").clamp(max=stored)
    near = torch.empty(F + (stored * F + n * K), device="cuda")      # (fp32 words: room for either type)
    near[:F] = a.reshape(-1)
    values = near[F:].view(dtype)
    values[:stored * F] = E[:stored].reshape(-1)
    got = []
    for dX, e, a_r in ((torch.empty(n, K, dtype=dtype, device="cuda"), E[:stored].contiguous(), a),
                       (values[stored * F:stored * F + n * K].view(n, K), values[:stored * F].view(stored, F), near[:F].view(H, D))):
        work = torch.empty(sar.sar_linear_workspace_bytes(n, K, F) // 4, device="cuda")
        dW = torch.zeros(K, F, device="cuda")
        sar.sar_linear_bwd_rows(X[:n], e if stored else None, rank.data_ptr() if stored else None, ds[:n], a_r, H, D, W, dW, dX, n,
                                dtype, work)
        got.append((dW, dX.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("K,H,D", [(64, 4, 16), (100, 4, 64), (72, 2, 50)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("where", ["X", "E", "W"])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38, 2.0 ** -111, 2.0 ** -126])
def test_values_that_are_not_split(K, H, D, dtype, where, value):
    """Infinities, NaN, values beyond bf16's largest and below its smallest piece: Z and dX as of many rows, bit for bit.
    (Whole tiles of 32 rows: fp32 dX is formed by another instruction for all rows of a tile in which one overflows.)"""
    X, E, W, _, _, _ = layer(K, H, D, dtype)
    {"X": X[70, 5:6], "E": E[70, 9:10], "W": W[11, 40:41]}[where].fill_(value)

    def run(n):
        Z, dX = torch.empty(n, H * D, dtype=dtype, device="cuda"), torch.empty(n, K, dtype=dtype, device="cuda")
        sar.sar_linear_fwd(X[:n], W, Z)
        sar.sar_linear_bwd(None, E[:n], W, None, dX, None)
        return Z, dX

    assert "k_few" in gu.kernels_of(lambda: run(96)) and "k_few" not in gu.kernels_of(lambda: run(MANY))
    for few, many in zip(run(96), run(MANY)):
        assert torch.equal(torch.isnan(few), torch.isnan(many[:96]))
        assert torch.equal(few.float().nan_to_num(7.0, 1.0, -1.0), many[:96].float().nan_to_num(7.0, 1.0, -1.0))


LINES = [  # rows, K, F, what is wanted, taken by the kernels of few rows; lines by dZ's columns and by the products wanted
    (torch.float32, 10_240, 128, 256, "both", True), (torch.float32, 10_240, 128, 260, "both", False),
    (torch.float32, 8_192, 128, 260, "both", True), (torch.bfloat16, 8_192, 256, 400, "both", True),
    (torch.bfloat16, 8_192, 256, 408, "both", False), (torch.bfloat16, 4_096, 256, 408, "both", True),
    (torch.float32, 10_240, 128, 32, "dX", True), (torch.float32, 10_240, 128, 36, "dX", False),
    (torch.float32, 8_192, 128, 36, "dX", True), (torch.float32, 8_192, 32, 36, "dX", True),
    (torch.float32, 8_000, 32, 36, "dX", False), (torch.float32, 100, 32, 32, "dX", True),
    (torch.float32, 100, 32, 1_028, "dX", True), (torch.bfloat16, 65_536, 32, 63, "dX", True),
    (torch.bfloat16, 65_536, 32, 64, "dX", False), (torch.bfloat16, 32_768, 32, 400, "dX", True),
    (torch.bfloat16, 32_768, 32, 408, "dX", False), (torch.bfloat16, 100, 16, 1_032, "dX", True),
    (torch.bfloat16, 8_192, 256, 128, "dX", True), (torch.bfloat16, 16_384, 128, 136, "dX", True),
    (torch.bfloat16, 32_768, 64, 136, "dX", False), (torch.bfloat16, 16_384, 64, 136, "dX", True),
    (torch.bfloat16, 2_048, 1_024, 256, "dX", False), (torch.bfloat16, 16_384, 64, 520, "dX", True),
    (torch.bfloat16, 12_288, 64, 520, "dX", False), (torch.bfloat16, 6_500, 64, 512, "dX", True),
    (torch.float32, 20_480, 64, 256, "dW", True), (torch.float32, 10_240, 128, 400, "dW", False),
    (torch.bfloat16, 49_152, 32, 400, "dW", False), (torch.bfloat16, 2_848, 256, 1_024, "dW", True),
    (torch.float32, 1_000, 516, 128, "Z", False), (torch.float32, 1_000, 516, 130, "Z", True),
    (torch.bfloat16, 1_000, 520, 128, "Z", False), (torch.bfloat16, 1_000, 512, 128, "Z", True),
    (torch.bfloat16, 8_192, 256, 32, "Z", True), (torch.bfloat16, 8_000, 256, 32, "Z", False),
    (torch.bfloat16, 8_192, 264, 32, "Z", False), (torch.bfloat16, 100, 64, 32, "Z", True),
    (torch.bfloat16, 2_432, 512, 400, "Z", True), (torch.bfloat16, 2_496, 512, 400, "Z", False)]


@pytest.mark.parametrize("dtype,n,K,F,what,few", LINES)
def test_both_sides_of_a_line(dtype, n, K, F, what, few):
    g = torch.Generator(device="cuda").manual_seed(n + K + F)
    draw = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
    X, dZ, W = draw(n, K).to(dtype), draw(n, F).to(dtype), draw(K, F) / K ** 0.5
    Z, dX, dW = torch.empty_like(dZ), torch.empty_like(X), torch.zeros(K, F, device="cuda")
    work = torch.empty(sar.sar_linear_workspace_bytes(n, K, F) // 4, device="cuda")
    x, d, w = X.double(), dZ.double(), W.double()
    if what == "Z":
        run, results = lambda: sar.sar_linear_fwd(X, W, Z), [(Z, x @ w, K)]
    else:
        run = lambda: sar.sar_linear_bwd(X, dZ, W, None if what == "dX" else dW, None if what == "dW" else dX, work)
        results = [(dX, d @ w.T, F)] * (what != "dW") + [(dW, x.T @ d, n)] * (what != "dX")
    assert ("k_few" in gu.kernels_of(run)) == few
    dW.zero_()
    run()
    for got, want, length in results:      # (stored bf16: half a unit of the value; sums as above, at most 32 rows' and their sums')
        tol = 2.0 ** -8 if got.dtype == torch.bfloat16 else max(2.0, min(length, 1024) ** 0.5) * 2.0 ** -24
        assert float((got.double() - want).norm() / want.norm()) < tol
