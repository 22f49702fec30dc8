"""The linear transform and its backward at the widths where their tiles end: contractions that are no
whole number of 16-byte pieces, narrow and wide weight gradients, rows that start at any element."""
import pytest
import torch

from oracle import sar_oracle as orc
from tests import gpu_util as gu
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu
f64 = lambda t: t.to(torch.float64).cpu().numpy()


SHAPES = [(3, 5), (7, 64), (9, 65), (32, 47), (33, 128), (61, 129), (100, 256), (129, 31),
          (200, 257), (255, 40), (257, 1), (400, 400), (47, 511), (512, 512), (5, 300), (1, 700)]


@pytest.mark.parametrize("K,F", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n", [1, 31, 700, 5003])
def test_shapes(K, F, dtype, n):
    check(K, F, dtype, n)


@pytest.mark.parametrize("K,F", [(400, 300), (354, 353), (512, 224), (330, 289)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_wide_column_slabs_of_many_rows(K, F, dtype):
    check(K, F, dtype, 20_011)


def check(K, F, dtype, n):
    g = torch.Generator().manual_seed(n + 1000 * K + F)
    # one element past an allocation's start: no row is aligned to more than that
    off = lambda n, w: torch.randn(n * w + 1, generator=g).to(dtype).cuda()[1:].view(n, w)
    X, dZ = off(n, K), off(n, F)
    W = (torch.randn(K, F, generator=g) / K ** 0.5).cuda()
    dW = torch.zeros(K, F, device="cuda")
    tol = 1e-5 if dtype == torch.float32 else 1e-2
    Z = gu.linear_fwd(X, W)[0]
    assert rel_err(f64(Z), orc.linear_fwd(f64(X), f64(W))) < tol
    dX = gu.linear_bwd(X, dZ, W, dW)
    want_dW, want_dX = orc.linear_bwd(f64(X), f64(dZ), f64(W))
    assert rel_err(f64(dX), want_dX) < tol
    assert rel_err(f64(dW), want_dW) < tol


@pytest.mark.parametrize("K,F", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_shapes_of_many_rows(K, F, dtype):
    """The same widths with more rows than the kernels of few rows take."""
    n = 70_001
    g = torch.Generator(device="cuda").manual_seed(1000 * K + F)
    off = lambda n, w: torch.randn(n * w + 1, generator=g, device="cuda").to(dtype)[1:].view(n, w)
    X, dZ = off(n, K), off(n, F)
    W = torch.randn(K, F, generator=g, device="cuda") / K ** 0.5
    dW, got = torch.zeros(K, F, device="cuda"), []

    def run():
        got[:] = gu.linear_fwd(X, W)[0], gu.linear_bwd(X, dZ, W, dW)

    assert "k_few" not in gu.kernels_of(run)
    dW.zero_()
    run()
    x, d, w = X.double(), dZ.double(), W.double()
    for have, want in zip(got + [dW], (x @ w, d @ w.T, x.T @ d)):
        assert float((have.double() - want).norm() / want.norm()) < (1e-5 if dtype == torch.float32 else 1e-2)
