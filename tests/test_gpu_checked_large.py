"""The kernels of the larger sizes through the checked library: the matrix forms of
distances and triplets, whole runs of packed triplets, contacts counted from
lists and from the tiles.  Sizes just above where each begins, ragged, results at
odd 4-byte offsets, every map: no map leaves the simplex, no unmasked store does,
nothing is written outside the result, and the values are the plain library's."""
import math

import numpy as np
import pytest
import torch

import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

MAPS = ["lambda", "bbox", "linear", "lambda_below", "recursive", "recursive_launch"]
PAD = -7.0


@pytest.fixture(scope="module", autouse=True)
def plain_library_after():
    yield
    smx.select_library(checked=False)


def _checked(f):
    """f() through the checked library, which must raise no flag."""
    smx.select_library(checked=True)
    try:
        smx.check_flags(clear=True)
        out = f()
        assert smx.check_flags(clear=True) == 0
        return out
    finally:
        smx.select_library(checked=False)


def _into(size, shift, f):
    """f(out) into a guarded buffer, `shift` floats past an allocation's start."""
    buf = torch.full((size + 64,), PAD, device="cuda")
    f(buf[shift:shift + size])
    assert (buf[:shift] == PAD).all() and (buf[shift + size:] == PAD).all()
    return buf[shift:shift + size]


@pytest.mark.parametrize("kind", MAPS)
@pytest.mark.parametrize("n,d,shift", [(5121, 66, 1), (8193, 37, 31)])
def test_distances(kind, n, d, shift):
    print(f"checked edm {kind} n={n} d={d}", flush=True)
    X = synth.normal(n, d, seed=n)
    X[n - 40:] = X[:40] + np.float32(1e-3)  # near pairs in few passes,
    X[1024:1280] = X[1024] + np.float32(1e-3) * X[1024:1280]  # and passes full of them
    X = torch.from_numpy(X).cuda()
    ref = smx.edm_packed(X)
    m = n * (n + 1) // 2
    assert torch.equal(_into(m, shift, lambda o: _checked(lambda: smx.edm_packed(X, kind, out=o))), ref)
    got, st = _checked(lambda: smx.edm_packed(X, kind, stats=True))
    assert torch.equal(got, ref) and int(st[0]) == m


@pytest.mark.parametrize("kind", MAPS)
def test_triplets(kind):
    print(f"checked triplets {kind}", flush=True)
    n = 1057
    P = torch.from_numpy(synth.rsa(n, seed=4, side=20.0 * (n / 8192) ** (1 / 3), dmin=0.8)).cuda()
    pot = smx.Pot(nu=1.0, at=True, lj=True)
    E0, G0 = smx.triplet_energy_grad(P, pot)
    E, G = _checked(lambda: smx.triplet_energy_grad(P, pot, kind))
    E1 = _checked(lambda: smx.triplet_energy(P, pot, kind))
    for e in (E, E1):
        assert (e - E0).abs().max() <= 1e-5 * E0.abs().max()
    assert (G - G0).norm(dim=1).max() <= 1e-5 * G0.norm(dim=1).max()


@pytest.mark.parametrize("kind", MAPS)
@pytest.mark.parametrize("shift", [1, 30])
def test_packed_triplets(kind, shift):
    print(f"checked packed {kind} {shift}", flush=True)
    n = 835
    P = torch.from_numpy(synth.rsa(n, seed=5, side=20.0 * (n / 8192) ** (1 / 3), dmin=0.8)).cuda()
    ref = smx.triplet_packed(P)
    got = _into(math.comb(n, 3), shift, lambda o: _checked(lambda: smx.triplet_packed(P, 1.0, kind, out=o)))
    assert torch.equal(got, ref)


@pytest.mark.parametrize("kind", [m for m in MAPS if m != "lambda_below"])
@pytest.mark.parametrize("n,rc", [(300, 2.0), (1100, 2.0), (1100, 4.2)])
def test_contacts(kind, n, rc):
    print(f"checked contacts {kind} n={n} rc={rc}", flush=True)
    C = torch.from_numpy(synth.uniform(n, 3, seed=6) * np.float32(n ** (1 / 3))).cuda()
    ref, _ = smx.quad_contacts(C, rc, stats=True)
    assert int(_checked(lambda: smx.quad_contacts(C, rc, kind)).item()) == int(ref.item())
