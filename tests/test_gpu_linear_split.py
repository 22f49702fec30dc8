"""The backward products of fp32 layers as sums of bf16 pieces: their error against 64-bit sums at the edges of the
tiles, and operands that have no such pieces (infinities, NaN, the largest finite values)."""
import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def backward(X, dZ, W):
    n, K = X.shape
    F = dZ.shape[1]
    work = torch.empty(max(1, sar.sar_linear_workspace_bytes(n, K, F) // 4), device="cuda")
    dW = torch.zeros(K, F, device="cuda")
    dX = torch.full((n, K), float("nan"), device="cuda")
    sar.sar_linear_bwd(X, dZ, W, dW, dX, work)
    return dW, dX


def operands(n, K, F, seed):
    g = torch.Generator().manual_seed(seed)
    draw = lambda *shape: torch.randn(*shape, generator=g).cuda()
    return draw(n, K), draw(n, F), draw(K, F)


# Column tiles 2, 4, 5 .. 8 and two slabs of dX (K), one and several steps that end inside a piece (F), last row blocks of
# 1, 127 and 128 rows, one slab of dW and many, its three widths, one chunk and chunks of fewer than 8 rows.
@pytest.mark.parametrize("n,K,F", [(1, 40, 17), (33, 31, 47), (129, 64, 64), (255, 100, 65), (4100, 128, 130),
                                   (30_000, 160, 100), (26_000, 190, 33), (26_011, 224, 257), (60_001, 256, 128),
                                   (50_000, 300, 60)])
def test_sums_against_64_bits(n, K, F):
    """A result of L products carries the rounding of its 6 L / 16 additions, each below 2^-24 of the running sum (at most
    the result's scale in its root mean square), and the left-out products, below 2^-23 of a product: sqrt(L) 2^-24 of
    the result with room for the rows' own spread.  (Measured: 0.9e-7 to 3e-7 of the result.)"""
    X, dZ, W = operands(n, K, F, seed=n + K)
    dW, dX = backward(X, dZ, W)
    for got, want, length in ((dX, dZ.double() @ W.double().T, F), (dW, X.double().T @ dZ.double(), n)):
        err = float((got.double() - want).norm() / want.norm())
        assert err < max(2.0, min(length, 1024) ** 0.5) * 2.0 ** -24, err


@pytest.mark.parametrize("length", [1, 2, 3, 5, 9, 15, 16, 17, 31, 33, 100, 257, 400, 2000, 6000])
@pytest.mark.parametrize("kind", ["normal", "uniform"])
def test_no_further_off_than_the_fp32_instruction(length, kind):
    """The forward product forms the same sums with the fp32 instruction: dW = (X^T) dZ over `length` rows and, from 17
    products on, dX = dZ (W^T).  (One and two rows: the same instruction, so the same error but for the order of two.)"""
    def pair(n, K, F):
        X, dZ, W = operands(n, K, F, seed=length)
        return (X, dZ, W) if kind == "normal" else tuple(torch.special.ndtr(t) for t in (X, dZ, W))

    def off(got, want):
        return float((got.double() - want).norm() / want.norm())

    X, dZ, _ = pair(length, 200, 100)
    dW, by_fp32 = torch.zeros(200, 100, device="cuda"), torch.empty(200, 100, device="cuda")
    work = torch.empty(sar.sar_linear_workspace_bytes(length, 200, 100) // 4, device="cuda")
    sar.sar_linear_bwd(X, dZ, None, dW, None, work)
    sar.sar_linear_fwd(X.T.contiguous(), dZ, by_fp32)
    want = X.double().T @ dZ.double()
    assert off(dW, want) <= 1.02 * off(by_fp32, want)
    for n in (3000, 12_000) if length > 16 else ():      # (few rows and many)
        _, dZ, W = pair(n, 100, length)
        dX, by_fp32 = torch.empty(n, 100, device="cuda"), torch.empty(n, 100, device="cuda")
        sar.sar_linear_bwd(None, dZ, W, None, dX, None)
        sar.sar_linear_fwd(dZ, W.T.contiguous(), by_fp32)
        want = dZ.double() @ W.double().T
        assert off(dX, want) <= 1.02 * off(by_fp32, want)


def test_sums_of_many_rows_lean_to_no_side():
    """The matrix cores cut small terms downwards; over a million rows the sums must not drift (the mean error of all
    entries, which independent roundings bring to 1/64 of their size)."""
    X, dZ, W = operands(1_000_000, 64, 64, seed=5)
    dW, _ = backward(X, dZ, W)
    d = dW.double() - X.double().T @ dZ.double()
    assert abs(float(d.mean())) < 0.1 * float(d.std())


@pytest.mark.parametrize("F", [17, 64, 256, 400])
@pytest.mark.parametrize("kind", ["normal", "uniform"])
def test_rows_of_errors_lean_to_no_side(F, kind):
    """dX is the next layer's error and is summed over all nodes there: its mean error, over all of it and over each
    column, is what independent roundings leave, 1/2500 and 1/316 of their size (ten and six of which are allowed)."""
    X, dZ, W = operands(100_000, 64, F, seed=9)
    if kind == "uniform":
        dZ, W = (torch.special.ndtr(t) for t in (dZ, W))
    _, dX = backward(X, dZ, W)
    d = dX.double() - dZ.double() @ W.double().T
    assert abs(float(d.mean())) < 10 / 2500 * float(d.std())
    assert float((d.mean(0) / d.std(0)).abs().max()) < 6 / 316


@pytest.mark.parametrize("n,K,F", [(300, 100, 64), (2_000, 256, 100), (700, 61, 47),
                                   (12_000, 100, 64), (6_000, 256, 100), (21_000, 61, 47)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
@pytest.mark.parametrize("where", ["X", "dZ", "W"])
def test_values_without_pieces(n, K, F, value, where):
    """One such value in an operand reaches the results it is a factor of, as in fp32 products, and no other."""
    X, dZ, W = operands(n, K, F, seed=F)
    if value == 3.4e38:                      # (beyond bf16's largest value; the products stay finite)
        X, dZ, W = X * 0.01, dZ * 0.01, W * 0.01
    row, col = n - 2, 19
    {"X": X, "dZ": dZ, "W": W}[where][row if where != "W" else K - 1, col] = value
    dW, dX = backward(X, dZ, W)
    for got, want in ((dX, dZ.double() @ W.double().T), (dW, X.double().T @ dZ.double())):
        finite = torch.isfinite(want)
        assert torch.equal(torch.isfinite(got), finite)
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(got[torch.isinf(got)].sign().double(), want[torch.isinf(want)].sign())
        w, e = want[finite], (got[finite].double() - want[finite]).abs()
        assert (e <= 1e-5 * torch.maximum(w.abs(), w.abs().median())).all()


@pytest.mark.parametrize("n,K,F", [(300, 100, 64), (700, 61, 47), (26_000, 256, 40)])
@pytest.mark.parametrize("exponent", [-111, -118, -126, -140])
@pytest.mark.parametrize("where", ["X", "dZ", "W", "one value of dZ"])
def test_small_values(n, K, F, exponent, where):
    """Operands whose last bits lie below bf16's smallest value: as close as larger ones, but for the roundings of `length`
    additions to fp32's smallest value, 2^-149, however small the result: each within half of it, 0.29 of it in the mean,
    so sqrt(length) of it is 3.4 standard deviations of their walk.  (Measured with the fp32 instruction: 1.3e-7 of the
    result down to 2^-126.)"""
    X, dZ, W = operands(n, K, F, seed=F)
    if where == "one value of dZ":
        value = float(dZ[n - 2, 19])
        dZ.zero_()
        dZ[n - 2, 19] = value * 2.0 ** exponent
    else:
        {"X": X, "dZ": dZ, "W": W}[where].mul_(2.0 ** exponent)
    dW, dX = backward(X, dZ, W)
    for got, want, length in ((dX, dZ.double() @ W.double().T, F), (dW, X.double().T @ dZ.double(), n)):
        root = max(2.0, min(length, 1024) ** 0.5)
        err = float((got.double() - want).norm())
        assert err < root * 2.0 ** -24 * float(want.norm()) + 2.0 ** -149 * (length * want.numel()) ** 0.5, err


@pytest.mark.parametrize("n,K,F", [(300, 100, 64), (700, 61, 47), (26_000, 256, 40)])
@pytest.mark.parametrize("value", [1.7e38, -1.7e38])
def test_results_near_the_largest_value(n, K, F, value):
    """1.9963 rounds up to 2 in its first piece, and 2 x 1.7e38 to beyond 3.4028e38 before the other pieces bring it back."""
    X, dZ, W = (torch.zeros_like(t) for t in operands(n, K, F, seed=1))
    X[n - 2, 5], dZ[n - 2, 19], W[7, 19] = 1.9963, value * 1.0022, 1.9963
    dW, dX = backward(X, dZ, W)
    for got, want in ((dX, dZ.double() @ W.double().T), (dW, X.double().T @ dZ.double())):
        assert float(want.abs().max()) > 3.39e38
        # (one product: rounded once by the fp32 instruction)
        assert float(((got.double() - want) / want.abs().max()).abs().max()) <= 2.0 ** -24


@pytest.mark.parametrize("n,H,D", [(1, 4, 16), (1000, 4, 32), (3001, 5, 20), (40_000, 2, 64)])
@pytest.mark.parametrize("formed", [False, True])
def test_in_place(n, H, D, formed):
    """dX written over dZ (at these widths): the kernel whose wavefronts read whole rows before they store any of them."""
    F = H * D
    X, dZ, W = operands(n, F, F, seed=n)
    want = dZ.double() @ W.double().T
    if formed:
        ds, a_r = torch.randn(n, H, device="cuda"), torch.randn(H, D, device="cuda")
        want = (dZ.double() + (ds.double()[:, :, None] * a_r.double()).reshape(n, F)) @ W.double().T
        sar.sar_linear_bwd_rows(None, dZ, None, ds, a_r, H, D, W, None, dZ, n, torch.float32, None)
    else:
        sar.sar_linear_bwd(None, dZ, W, None, dZ, None)
    assert float((dZ.double() - want).norm() / want.norm()) < F ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("n,K,F", [(12_000, 100, 64), (6_000, 256, 100), (21_000, 61, 47), (6_000, 200, 100), (26_000, 256, 40)])
def test_sizes_above_that_many_rows_take(n, K, F):
    X, dZ, W = operands(n, K, F, seed=3)
    names = gu.kernels_of(lambda: backward(X, dZ, W))
    assert "k_dx_split" in names and "k_dw_split" in names
