"""4-point contacts counted from the contacts (calls without statistics, n >=
256), exact against the oracle: around the first size, at the edges of a 64-wide
word, of one, two and four words a lane, on both sides of the density at which
the device takes the tiles instead, and on every map."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

KINDS = ["lambda", "bbox", "linear", "recursive", "recursive_launch"]


def _cloud(n, seed):
    return synth.uniform(n, 3, seed=seed) * np.float32(n ** (1 / 3))


@pytest.mark.parametrize("n", [255, 256, 257, 320, 1023, 1024, 1025, 1088, 4096, 4097, 8192, 8200])
def test_sizes(n):
    X = _cloud(n, n)
    Xt = torch.from_numpy(X).cuda()
    for rc in (1.2, 2.1):
        print(f"rows n={n} rc={rc}", flush=True)
        assert int(smx.quad_contacts(Xt, rc).item()) == oracle.quad_contacts(X, rc)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [300, 1100])
def test_maps(kind, n):
    X = _cloud(n, 3)
    c = int(smx.quad_contacts(torch.from_numpy(X).cuda(), 2.0, kind).item())
    assert c == oracle.quad_contacts(X, 2.0) > 0


@pytest.mark.parametrize("n,rc", [(300, 1e3), (1024, 1e3), (1025, 1e3), (1100, 3.0), (1100, 2.4), (1100, 0.0)])
def test_dense_and_empty(n, rc):
    """All pairs in contact (always by rows up to n = 1024, by tiles above), a
    degree over and under the switch (64 at n = 1100), and none."""
    X = _cloud(n, 17)
    ref = math.comb(n, 4) if rc > 100 else oracle.quad_contacts(X, rc)
    assert int(smx.quad_contacts(torch.from_numpy(X).cuda(), rc).item()) == ref


def test_workspace_contents_do_not_matter():
    """Words below a row's own tile are never written, so whatever the workspace
    held there must not reach the count."""
    n = 700
    X = _cloud(n, 4)
    Xt = torch.from_numpy(X).cuda()
    ref = oracle.quad_contacts(X, 1.9)
    for fill in (0, 255):
        ws = torch.full((smx.workspace_bytes(3, n),), fill, dtype=torch.uint8, device="cuda")
        assert int(smx.quad_contacts(Xt, 1.9, ws=ws).item()) == ref
