"""The builder's grouping of pairs at the lengths where its sorts change, with rows too long for a bucket,
and restricted handles of it: index arrays bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import sar_oracle as orc
from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# rows of 16 lanes, of one, two and four values per lane, of merged pieces, of a network in LDS and in memory
LENGTHS = [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1025, 4095, 4096, 4097, 8192, 8193, 20000]


def check(b, want):
    for q, w in enumerate(want):
        v = gu.view_arrays(b, q)
        for name in ("indptr", "indices", "t_indptr", "t_indices"):
            assert np.array_equal(v[name], getattr(w, name).astype(np.int32)), (q, name)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("n_extra", [0, 60_000])        # alone, and among many short rows
@pytest.mark.parametrize("idx_dtype", [torch.int32, torch.int64])
def test_row_lengths(transposed, n_extra, idx_dtype):
    rng = np.random.default_rng(5)
    N, P = 40_000, 2
    part = (np.arange(N) % P).astype(np.int32)
    own = np.flatnonzero(part == 0)
    hub = np.repeat(own[3 * np.arange(len(LENGTHS))], LENGTHS)
    other = own[rng.integers(0, own.size, hub.size)]      # repeated pairs among them
    a, b = (other, hub) if transposed else (hub, other)
    dst = np.concatenate([a, own[rng.integers(0, own.size, n_extra)]])
    src = np.concatenate([b, rng.integers(0, N, n_extra)])
    order = rng.permutation(dst.size)
    src, dst = src[order], dst[order]
    want, _ = orc.build_blocks(src, dst, part, P, 0)
    h = gu.build_blocks(src, dst, part, P, 0, idx_dtype=idx_dtype)
    check(h, want)
    ids = rng.integers(0, h.n_dst, 500).astype(np.int32)
    sub = sar.sar_blocks_subset(h, torch.from_numpy(ids).cuda())
    check(sub, orc.subset_blocks(want, ids)[0])
    h.close()                                             # the restricted handle is independent of it
    again = gu.build_blocks(src, dst, part, P, 0, idx_dtype=idx_dtype)     # on memory the first one gave up
    check(again, want)
    check(sub, orc.subset_blocks(want, ids)[0])


def test_many_rows_too_long_for_a_bucket():
    """More shares of listed buckets than the sort has workgroups, one long row in each bucket."""
    rng = np.random.default_rng(6)
    N, rows, each = 40_000, 100, 11_000
    part = np.zeros(N, dtype=np.int32)
    dst = np.repeat(rng.permutation(N)[:rows], each)
    src = rng.integers(0, N, dst.size)
    want, _ = orc.build_blocks(src, dst, part, 1, 0)
    h = gu.build_blocks(src, dst, part, 1, 0)
    check(h, want)
    h.close()
