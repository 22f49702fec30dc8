"""The builder's prefix sums where their tiles of 2048 values end, and beyond 4096 tiles, where the sums of the tiles are
scanned by a pass of their own: index arrays bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import sar_oracle as orc
from tests import gpu_util as gu
from tests.test_gpu_builder_rows import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_offsets", [2, 2047, 2048, 2049, 2055, 2 * 2048 + 1, 257 * 2048 + 3, 4096 * 2048, 4096 * 2048 + 1])
def test_offsets_of_rows(n_offsets):
    rng = np.random.default_rng(n_offsets)
    N = n_offsets - 1
    E = 6_000
    dst = np.concatenate([rng.integers(0, N, E), [0, N - 1, N - 1]])
    src = np.concatenate([rng.integers(0, N, E), [N - 1, 0, N - 1]])
    part = np.zeros(N, dtype=np.int32)
    want, _ = orc.build_blocks(src, dst, part, 1, 0)
    h = gu.build_blocks(src, dst, part, 1, 0)
    check(h, want)
    h.close()
