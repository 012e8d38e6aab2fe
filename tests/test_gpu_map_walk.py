"""The element walk of the map dumps at the edges of its launch shapes: one wave or
256 threads a block (tiles of 1024 and 4096 elements, parallel spaces either side
of 8192 blocks), fewer outer coordinates than threads, and ragged last tiles.
Ids are a bijection onto [0, V), so the checksum is that of 0 .. V - 1, exactly.
"""
import math

import numpy as np
import pytest
import torch

import paper_1610_07394_amd as smx

pytestmark = pytest.mark.gpu


def _checksum(v):
    total = np.uint64(0)
    with np.errstate(over="ignore"):
        for lo in range(0, v, 1 << 22):
            z = np.arange(lo, min(v, lo + (1 << 22)), dtype=np.uint64) + np.uint64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            total += (z ^ (z >> np.uint64(31))).sum(dtype=np.uint64)
    return int(total.astype(np.int64))


@pytest.mark.parametrize("m,n,rho", [
    (2, 130, 1), (2, 333, 2), (2, 1001, 16), (2, 1023, 32), (2, 1000, 64), (2, 8190, 64), (2, 1500, 128),
    (3, 17, 1), (3, 65, 2), (3, 130, 4), (3, 203, 8), (3, 250, 16), (3, 417, 16), (3, 100, 32),
    (4, 9, 1), (4, 21, 2), (4, 50, 4), (4, 60, 8), (4, 131, 8), (4, 40, 16)])
@pytest.mark.parametrize("strict", [True, False])
def test_counts_and_checksums(m, n, rho, strict):
    f = {2: smx.simplex_map2, 3: smx.simplex_map3, 4: smx.simplex_map4}[m]
    v = math.comb(n if strict else n + m - 1, m)
    want = _checksum(v)
    for kind in ("lambda", "linear", "bbox", "recursive"):
        st = f(n, rho, kind, strict=strict, tiles=True, stats=True)[1].tolist()
        assert st[:2] == [v, want], (kind, st)
        assert st[2] == math.comb(-(-n // rho) + m - 1, m)
