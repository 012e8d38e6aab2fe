"""Workspace sizes of the triplet calls by potential, mode and limit (host only)."""
import ctypes

import pytest

import paper_1610_07394_amd as smx

AT, LJ = smx.Pot(at=True, lj=False), smx.Pot(at=False, lj=True)


def _least(n):
    return (3 * 32768 + 24 * n + 255) // 256 * 256


@pytest.mark.parametrize("n", [0, 3, 767, 768, 1023, 1024, 8192, 1 << 18, (1 << 18) + 1, 1 << 20])
def test_only_the_calls_that_use_it_ask_for_more(n):
    most = smx.workspace_bytes(2, n)
    for pot in (AT, LJ, smx.Pot(lj=True)):
        for grad in (False, True):
            for stats in (False, True):
                size = smx.triplet_workspace_bytes(n, pot, grad, stats)
                matrix = pot.at and not stats and (768 if grad else 1024) <= n <= 1 << 18
                assert size == (most if matrix else _least(n))


@pytest.mark.parametrize("n", [1024, 5000, 8192, 30000, 100000])
def test_limits(n):
    """Every smaller limit gets a plan that fits it, down to the least."""
    size, seen = smx.triplet_workspace_bytes(n, AT), []
    while size > _least(n):
        seen.append(size)
        assert smx.triplet_workspace_bytes(n, AT, limit=size) == size
        size = smx.triplet_workspace_bytes(n, AT, limit=size - 1)
        assert size < seen[-1]
        if len(seen) > 4:  # then fewer columns of one form, 256 by 256
            size = smx.triplet_workspace_bytes(n, AT, limit=size // 2)
    assert len(seen) >= 3 and size == _least(n)
    assert smx.triplet_workspace_bytes(n, AT, limit=0) == _least(n)


def test_bad_arguments():
    L = smx.lib()
    c = AT._c()
    assert L.smx_triplet_workspace_bytes(-1, ctypes.byref(c), 1, 0, 1 << 40) == 0
    assert L.smx_triplet_workspace_bytes(100, None, 1, 0, 1 << 40) == 0
