"""Packed triplet energies over FP32's range: elements that are ordinary numbers
though a factor of them is not (k far from a close pair, a large or small nu), by
both kernels, against the definition in FP64.

The bar is 1e-5 of an element's own scale nu / (r r r)^3, as for every packed energy.
"""
import math

import numpy as np
import pytest
import torch

import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu


def _check(X, nu):
    """Every element whose scale is a normal FP32 number with room for its last bits."""
    n = len(X)
    x = torch.from_numpy(X).cuda().double()
    got = smx.triplet_packed(x.float(), nu).double()
    i, j, k = torch.combinations(torch.arange(n, device="cuda"), 3).T
    a, b, c = x[j] - x[i], x[k] - x[j], x[k] - x[i]
    ra, rb, rc = (v.norm(dim=1) for v in (a, b, c))
    cosines = ((a * b).sum(1) / (ra * rb)) * ((b * c).sum(1) / (rb * rc)) * ((a * c).sum(1) / (ra * rc))
    scale = nu / (ra * rb * rc) ** 3
    normal = (scale.abs() > 1e-36) & (scale.abs() < 1e38)
    assert normal.any()
    err = ((got - scale * (1 - 3 * cosines)) / scale).abs()[normal]
    print(f"n={n} nu={nu:g}: {int(normal.sum())} of {len(got)} elements, error {err.max().item():.1e}", flush=True)
    assert err.max().item() <= 1e-5


# 40 particles are the tile kernel's, 710 with whole runs; the test takes 150 of them
def _far(n, close, far, seed):
    r = np.random.default_rng(seed)
    X = r.standard_normal((n, 3))
    X = X / np.linalg.norm(X, axis=1, keepdims=True) * far * (1 + r.random((n, 1)))
    X[1] = X[0] = 0
    X[1, 0] = close
    return X.astype(np.float32)


@pytest.mark.parametrize("close,far", [(1e-3, 1e7), (0.1, 3e6), (1.0, 1e3)])
def test_far_third_particle(close, far):
    _check(_far(60, close, far, 1), 1.0)


@pytest.mark.parametrize("nu,close,far", [(1e30, 1e-3, 1e3), (-1e30, 1e-3, 1e3), (3e38, 1e-2, 1e4), (1e-30, 1e-3, 1.0),
                                          (1e-37, 1.0, 1.5), (0.7, 0.5, 2.0)])
def test_nu(nu, close, far):
    X = _far(60, close, far, 2)
    X[[1, 30]] = X[[30, 1]]  # the close pair as (i, k) too
    _check(X, float(np.float32(nu)))


def test_whole_runs_keep_the_tile_kernels_values():
    X = torch.from_numpy(np.concatenate((_far(400, 1e-3, 1e7, 3), synth.uniform(310, 3, seed=3)))).cuda()
    for nu in (1.0, 1e30, -2.5e-30):
        got, ref = smx.triplet_packed(X, nu), smx.triplet_packed(X, nu, stats=True)[0]
        assert torch.equal(torch.nan_to_num(got, nan=7.0), torch.nan_to_num(ref, nan=7.0))
    assert smx.triplet_packed(X, 0.0).abs().max().item() == 0.0
    assert got.numel() == math.comb(710, 3)
