"""The builder's sorts of short groups, alone and side by side in a wavefront, and its launch lists where a workgroup
places more rows than once: index arrays and lists against the oracle."""
import numpy as np
import pytest
import torch

from oracle import sar_oracle as orc
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def check(src, dst, part, P):
    want, _ = orc.build_blocks(src, dst, part, P, 0)
    b = gu.build_blocks(src, dst, part, P, 0)
    for q, w in enumerate(want):
        v = gu.view_arrays(b, q)
        for name in ("indptr", "indices", "t_indptr", "t_indices"):
            assert np.array_equal(v[name], getattr(w, name).astype(np.int32)), (q, name)
        for rows, ptr in ((v["rows"], w.indptr), (v["t_rows"], w.t_indptr)):
            deg = np.diff(ptr)
            assert sorted(rows.tolist()) == np.flatnonzero(deg > 0).tolist()
            cls = np.floor(np.log2(deg[rows]))
            assert np.all(np.diff(cls) <= 0)
            assert np.all(np.diff(rows)[np.diff(cls) == 0] > 0)      # in a class by id
    b.close()


# 8 lanes, 16 lanes, a wavefront with one, two and four values a lane; all values equal, few of them, all different
@pytest.mark.parametrize("lengths", [range(1, 9), range(7, 18), [8] * 40, [16, 9, 1] * 20, range(17, 66), [100, 128, 129, 255, 256, 257]])
@pytest.mark.parametrize("values", [1, 3, 4_000])
@pytest.mark.parametrize("order", ["ascending", "descending", "mixed"])
def test_groups(lengths, values, order):
    lengths = np.array(list(lengths) * 3)
    rng = np.random.default_rng(int(lengths.sum()) + values)
    N = 4_000
    dst = np.repeat(rng.permutation(N)[:lengths.size], lengths)
    src = rng.integers(0, values, dst.size)
    by = {"ascending": np.argsort(src, kind="stable"), "descending": np.argsort(-src, kind="stable"),
          "mixed": rng.permutation(dst.size)}[order]
    check(src[by], dst[by], np.zeros(N, dtype=np.int32), 1)


@pytest.mark.parametrize("n", [2_047, 2_048, 2_049, 9_000])
def test_lists_of_many_rows(n):
    rng = np.random.default_rng(n)
    part = (np.arange(2 * n) % 2).astype(np.int32)
    dst = 2 * rng.integers(0, n, 3 * n)
    check(rng.integers(0, 2 * n, dst.size), dst, part, 2)


@pytest.mark.parametrize("sizes", [[6_000, 0, 1, 4_096, 0, 0, 2_049, 1], [1, 0, 9_000], [0, 0, 5, 2_048], [3] * 60 + [20_000]])
def test_lists_of_blocks_of_any_size(sizes):
    """Blocks of no source, of one, of whole and broken tiles, the destinations' own among them."""
    rng = np.random.default_rng(len(sizes))
    part = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    N, mine = part.size, np.flatnonzero(part == part[-1])
    part = (part - part[-1]) % len(sizes)                     # the last block's nodes are partition 0
    dst = mine[rng.integers(0, mine.size, 2 * N)]
    check(rng.integers(0, N, dst.size), dst, part.astype(np.int32), len(sizes))
