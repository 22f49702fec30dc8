"""Device memory that the library keeps between builder calls: bounded by the handles' life."""
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
    assert not [o for o in gc.get_objects() if isinstance(o, sar.Blocks) and o._h is not None]


def test_a_failed_build_of_the_only_handle_keeps_nothing():
    src, dst, part = edges(8_000_000, 100_000)
    src[-1] = 100_000                                    # out of range: found once the scratch has been taken
    no_other_handle()
    before = free_bytes()
    with pytest.raises(sar.SarError):
        sar.sar_blocks_build(src, dst, part, 1, 0, sar.SAR_BUILD_TRANSPOSE)
    assert before - free_bytes() < 4 * MB
