"""The workspace that a handle needs, in bytes: callers hold sizes from earlier builds, so
what was enough stays enough.  Memory for the draws of baths ahead of the steps is apart."""
from __future__ import annotations

import pytest

from paper_1907_10514_amd import lion


@pytest.mark.parametrize("n,traps,need", [
    (1, 1, (495104, 560640)), (8, 1, (495104, 560640)), (100, 1, (519680, 585216)),
    (1024, 1, (863744, 929280)), (2048, 1, (2510848, 2641920)),
    (16384, 1, (32649728, 33698304)), (65536, 1, (432581888, 436776192)),
    (200000, 1, (399933696, 412778752)), (5120, 256, (907264, 907264)),
    (131072, 512, (22672896, 22672896)), (1048576, 4096, (181372416, 181372416))])
def test_need_does_not_grow(n, traps, need):
    for prec, most in ((0, need[0]), (1, need[1]), (2, need[1])):
        assert 0 < lion.lion_workspace_bytes(n, traps, prec) <= most


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("n", [1, 64, 65, 1024, 16384, 65536, 109226, 131072, 10 ** 7])
def test_bath_memory_is_useful_or_none(n, batched):
    extra, row = lion.bath_memory_bytes(n, batched), 8 * ((n + 63) // 64 * 64)
    least, most = ((1 + 3 * 32) * row, 48 << 20) if batched else (10 * row, 16 << 20)
    assert extra == 0 or least <= extra <= most
    assert extra > 0 or least > most
