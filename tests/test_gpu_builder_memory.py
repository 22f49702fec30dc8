"""Device memory that the library keeps between builder calls: bounded by the handles' life, given back on request."""
import gc

import pytest
import torch

from paper_2111_06483_amd import sar
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
MB = 1 << 20


def edges(E, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    src, dst = (torch.randint(0, N, (E,), generator=g, device="cuda") for _ in range(2))
    return src, dst, torch.zeros(N, dtype=torch.int32, device="cuda")


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def no_other_handle(but=None):
    gc.collect()
    assert not [o for o in gc.get_objects() if type(o) is sar.Blocks and o._h is not None and o is not but]


def test_a_failed_build_of_the_only_handle_keeps_nothing():
    src, dst, part = edges(8_000_000, 100_000)
    src[-1] = 100_000                                    # out of range: found once the scratch has been taken
    no_other_handle()
    before = free_bytes()
    with pytest.raises(sar.SarError):
        sar.sar_blocks_build(src, dst, part, 1, 0, sar.SAR_BUILD_TRANSPOSE)
    assert before - free_bytes() < 4 * MB


def test_idle_memory_is_released_on_request():
    src, dst, part = edges(8_000_000, 100_000)
    no_other_handle()
    small = sar.sar_blocks_build(src[:1000], dst[:1000], part, 1, 0, 0)
    before = free_bytes()
    sar.sar_blocks_build(src, dst, part, 1, 0, sar.SAR_BUILD_TRANSPOSE).close()
    kept = before - free_bytes()
    assert 32 * MB < kept <= 1024 * MB                   # the closed handle's arrays, while `small` lives
    sar.sar_release_memory()
    assert before - free_bytes() < 4 * MB
    assert sar.sar_blocks_degree(small) is not None      # the living handle is untouched
    small.close()


def index_arrays(b):
    out = []
    for q in range(b.P):
        v = b.view(q)
        for ptr, n in ((v.indptr, v.n_dst + 1), (v.indices, v.nnz), (v.t_indptr, v.n_src + 1), (v.t_indices, v.nnz)):
            if ptr:
                out.append(sar.device_array(ptr, int(n)).clone())
    return out


class Full:
    """All of the device's memory but what room() leaves, and one handle."""

    def __init__(self, handle):
        self.handle = handle

    def __enter__(self):
        no_other_handle(self.handle)
        sar.sar_release_memory()
        torch.cuda.empty_cache()
        self.last = None
        self.most = torch.empty(free_bytes() - 1024 * MB, dtype=torch.uint8, device="cuda")
        lo, hi = 512, 4096             # the memory said to be free is less than what can be had
        while hi - lo > 4:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if self.take(mid) else (lo, mid)
        self.rest = lo
        return self

    def take(self, mb):
        self.last = None
        sar.sar_release_memory()
        torch.cuda.empty_cache()
        try:
            self.last = torch.empty(mb * MB, dtype=torch.uint8, device="cuda")
        except torch.cuda.OutOfMemoryError:
            return False
        return True

    def room(self, mb):
        assert self.take(self.rest - mb)

    def __exit__(self, *_):
        self.most = self.last = None
        torch.cuda.empty_cache()


def test_builds_with_little_room():
    """24 Mi edges: 192 MiB of what the counting pass may leave for the scatter, and 96 each of sources, pairs and derived
    indexes.  Memory that only speeds a build up is done without, and the arrays are the same; a build that does not fit
    says so and leaves no error for the next one.  (Beside a handle that lives: a device's only one leaves nothing.)"""
    fused = sar.SAR_BUILD_TRANSPOSE | sar.SAR_BUILD_FUSED
    src, dst, part = edges(24 * MB, 100_000)
    small = src.to(torch.int32), dst.to(torch.int32)
    cases = []
    # room for none of the first; for it but not the sources, nor the pairs, beside it; for all of these but not the derived ones
    for P, flags, room in ((8, sar.SAR_BUILD_TRANSPOSE, 150), (1, 0, 240), (1, 0, 320), (1, fused, 450)):
        part = torch.arange(100_000, device="cuda", dtype=torch.int32) % P
        b = sar.sar_blocks_build(src, dst, part, P, 0, flags)
        cases.append((P, flags, room, part, index_arrays(b)))
        b.close()
    living = sar.sar_blocks_build(src[:1000], dst[:1000], part, 1, 0, 0)
    with Full(living) as full:
        for P, flags, room, part, want in cases:
            for s, d in ((src, dst), small):
                full.room(room)
                b = sar.sar_blocks_build(s, d, part, P, 0, flags)
                full.last = None                         # (room for copies of its arrays)
                torch.cuda.empty_cache()
                got = index_arrays(b)
                b.close()
                assert len(got) == len(want) and all(torch.equal(x, y) for x, y in zip(got, want)), (P, flags, room)
                del got
        full.room(100)
        with pytest.raises(sar.SarError) as e:
            sar.sar_blocks_build(src, dst, part, 1, 0, 0)
        assert "hipMalloc" in str(e.value)
        sar.sar_blocks_build(src[:1000], dst[:1000], part, 1, 0, 0).close()
    living.close()


def test_edges_are_stored_where_the_memory_is_kept():
    """A device's only handle, or edges of more than 256 MiB in (key, value) pairs of 8 bytes: the memory would go to the driver
    and come from it again, which takes longer than gathering twice.  Both ways to the same arrays."""
    no_other_handle()
    most = 32 * MB                                        # edges
    src, dst, part = edges(most + 1, 100_000)
    part = torch.arange(100_000, device="cuda", dtype=torch.int32) % 16
    arrays = []
    for E, alive, stored in ((200_001, False, False), (200_001, True, True), (most, False, False), (most, True, True),
                             (most + 1, True, False)):
        other = sar.sar_blocks_build(src[:1000], dst[:1000], part, 16, 0, 0) if alive else None

        def build():
            b = sar.sar_blocks_build(src[:E], dst[:E], part, 16, 0, sar.SAR_BUILD_TRANSPOSE)
            arrays.append(index_arrays(b))
            b.close()

        names = [n for n in gu.kernels_of(build).split("\n") if "k_bucket_scatter" in n]
        assert len(names) == 1 and ("StoredEdges" in names[0]) == stored, (E, alive, names)
        if other:
            other.close()
    for x, y in (arrays[0:2], arrays[2:4]):
        assert all(torch.equal(a, b) for a, b in zip(x, y))


def test_keys_in_several_passes():
    """256 partitions and 2^20 + 1 rows: more (block, row) pairs than one pass groups; the scatter reads the edge list."""
    N, P, E = (1 << 20) + 256, 256, 400_000
    g = torch.Generator(device="cuda").manual_seed(2)
    part = torch.zeros(N, dtype=torch.int32, device="cuda")
    others = torch.randperm(N, generator=g, device="cuda")[:P - 1]
    part[others] = torch.arange(1, P, dtype=torch.int32, device="cuda")
    src = torch.randint(0, N, (E,), generator=g, device="cuda")
    src[::3] = others[torch.randint(0, P - 1, (src[::3].numel(),), generator=g, device="cuda")]
    dst = torch.randint(0, N, (E,), generator=g, device="cuda")
    rank = torch.zeros(N, dtype=torch.int64, device="cuda")
    rank[part == 0] = torch.arange(int((part == 0).sum()), device="cuda")
    kept = part[dst] == 0
    q_of, i, j = part[src[kept]].long(), rank[dst[kept]], rank[src[kept]]       # (the others have one node each: rank 0)
    n_dst = int((part == 0).sum())
    b = sar.sar_blocks_build(src, dst, part, P, 0, 0)
    assert b.n_dst == n_dst == (1 << 20) + 1
    for q in range(P):
        v, mine = b.view(q), q_of == q
        key = torch.sort(i[mine] * N + j[mine])[0]
        assert v.nnz == key.numel()
        assert torch.equal(sar.device_array(v.indices, int(v.nnz)).long(), key % N)
        want = torch.zeros(n_dst + 1, dtype=torch.int64, device="cuda")
        want[1:] = torch.cumsum(torch.bincount(key // N, minlength=n_dst), 0)
        assert torch.equal(sar.device_array(v.indptr, n_dst + 1).long(), want)
    b.close()
