"""Scores that leave with bf16 rows: bit for bit those of a pass over the stored rows, and the rows those of a transform without
scores, at every way the heads lie in the tiles and slabs; shapes beside the line take the pass."""
import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# heads of one, two and four tiles; one head, heads that fill no power of two, more than one slab of columns
WITH_ROWS = [(8, 32), (1, 32), (5, 32), (16, 32), (4, 64), (3, 64), (1, 64), (9, 64), (2, 128), (1, 128), (3, 128)]
BY_A_PASS = [(1, 256), (2, 100), (4, 16), (8, 8), (1, 48)]


@pytest.mark.parametrize("H,D", WITH_ROWS + BY_A_PASS)
@pytest.mark.parametrize("K", [8, 100, 128, 131, 256])
@pytest.mark.parametrize("n", [70_001, 131_072])        # the last tile with one row, and whole
def test_scores_of_many_rows(H, D, K, n):
    g = torch.Generator(device="cuda").manual_seed(1000 * K + 10 * H + D + n)
    X = torch.randn(n, K, generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn(K, H * D, generator=g, device="cuda") / K ** 0.5
    a1, a2 = (torch.randn(H, D, generator=g, device="cuda") for _ in range(2))
    X[5, 3] = float("inf")
    rows = lambda: torch.full((n, H * D), 7.0, dtype=torch.bfloat16, device="cuda")
    half = lambda: torch.full((n, H), 7.0, device="cuda")
    bits = lambda t: t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)
    Z, want, w1, w2 = rows(), rows(), half(), half()
    sar.sar_linear_fwd(X, W, want)
    sar.sar_gat_scores(want.view(n, H, D), a1, w1)
    sar.sar_gat_scores(want.view(n, H, D), a2, w2)
    s1, s2, one = half(), half(), half()
    kernels = gu.kernels_of(lambda: sar.sar_linear_fwd(X, W, Z, a1, s1, a2, s2))
    # (more slabs than four go by steps; where the weights leave less than 2 KB of LDS the pass stays)
    with_rows = (H, D) in WITH_ROWS and not (K == 256 and H * D > 512) and not (K == 131 and H * D > 128)
    if (H, D) in BY_A_PASS:
        assert "k_scores" in kernels
    elif with_rows:
        assert "k_scores" not in kernels
    finite = torch.isfinite(want.float()).all(1)
    assert torch.equal(bits(Z)[finite], bits(want)[finite])
    for s, w in ((s1, w1), (s2, w2)):
        assert torch.equal(bits(s)[finite], bits(w)[finite])
        assert torch.equal(torch.isfinite(s), torch.isfinite(w))
    sar.sar_linear_fwd(X, W, Z, a2, one)                  # one vector alone
    assert torch.equal(bits(one)[finite], bits(w2)[finite])


# at the limits: weights that leave just room for the vectors' values beside them, or not; one slab of columns and several
@pytest.mark.parametrize("K,H,D,with_rows", [(256, 16, 32, True), (256, 8, 64, True), (256, 4, 128, True), (256, 9, 64, False),
                                             (256, 5, 128, False), (131, 4, 32, True), (131, 2, 64, True), (131, 8, 32, False),
                                             (131, 4, 64, False), (131, 3, 128, False), (512, 4, 64, True), (1024, 1, 32, True)])
@pytest.mark.parametrize("both", [False, True])
def test_which_scores_leave_with_the_rows(K, H, D, with_rows, both):
    n = 70_001
    X, W = torch.randn(n, K, device="cuda").to(torch.bfloat16), torch.randn(K, H * D, device="cuda")
    a, s, w = torch.randn(H, D, device="cuda"), torch.empty(n, H, device="cuda"), torch.empty(n, H, device="cuda")
    Z = torch.empty(n, H * D, dtype=torch.bfloat16, device="cuda")
    other = (a.neg(), torch.empty_like(s)) if both else ()
    kernels = gu.kernels_of(lambda: sar.sar_linear_fwd(X, W, Z, a, s, *other))
    assert ("k_scores" not in kernels) == with_rows
    sar.sar_gat_scores(Z.view(n, H, D), a, w)
    assert torch.equal(s, w) and (not both or torch.equal(other[1], -w))


def test_rows_that_begin_off_a_piece_are_refused_with_scores():
    """As by the pass over the stored rows, which reads them in 16-byte pieces."""
    n, K, H, D = 70_001, 64, 4, 64
    X, W = torch.randn(n, K, device="cuda").to(torch.bfloat16), torch.randn(K, H * D, device="cuda")
    Z = torch.empty(n * H * D + 4, dtype=torch.bfloat16, device="cuda")[4:].view(n, H * D)
    a, s = torch.randn(H, D, device="cuda"), torch.empty(n, H, device="cuda")
    with pytest.raises(sar.SarError, match="16-byte aligned") as e:
        sar.sar_linear_fwd(X, W, Z, a, s)
    assert e.value.code == sar.SAR_ERR_INVALID_ARG


@pytest.mark.parametrize("over", ["first", "last", "weights"])
@pytest.mark.parametrize("second", [False, True])
def test_scores_over_an_operand(over, second):
    """Scores may lie over the inputs or the weights: rows and scores are those of a call with memory of their own."""
    n, K, H, D = 70_001, 128, 8, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(n, K, generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn(K, H * D, generator=g, device="cuda") / K ** 0.5
    a1, a2 = (torch.randn(H, D, generator=g, device="cuda") for _ in range(2))
    want, w1, w2 = torch.empty(n, H * D, dtype=torch.bfloat16, device="cuda"), *(torch.empty(n, H, device="cuda") for _ in range(2))
    sar.sar_linear_fwd(X, W, want, a1, w1, a2, w2)
    Z, own = torch.empty_like(want), torch.empty(n, H, device="cuda")
    if over == "weights":
        room = torch.zeros(n * H, device="cuda")
        room[:W.numel()] = W.flatten()
        W, shared = room[:W.numel()].view(K, H * D), room.view(n, H)
    else:
        flat = X.flatten().view(torch.float32)
        shared = (flat[:n * H] if over == "first" else flat[-n * H:]).view(n, H)
    sar.sar_linear_fwd(X, W, Z, a1, own if second else shared, a2, shared if second else own)
    assert torch.equal(Z, want)
    s1, s2 = (own, shared) if second else (shared, own)
    assert torch.equal(s1, w1) and torch.equal(s2, w2)
