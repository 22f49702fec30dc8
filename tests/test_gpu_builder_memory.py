"""Device memory that the library keeps between builder calls: bounded by the handles' life, given back on request."""
import gc

import pytest
import torch

from paper_2111_06483_amd import sar

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


def no_other_handle():
    gc.collect()
    assert not [o for o in gc.get_objects() if type(o) is sar.Blocks and o._h is not None]


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
