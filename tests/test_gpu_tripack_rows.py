"""Packed triplet energies written run by run (n >= 704): bit for bit the tile
kernel's values (calls with statistics take it), at the first sizes, at the edges
of the 32-wide tiles and of the 224-element steps of a run, on every map, and into
buffers at any 4-byte offset from a 128-byte line, whose neighbours stay intact."""
import math

import numpy as np
import pytest
import torch

import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

KINDS = ["lambda", "bbox", "linear", "lambda_below", "recursive", "recursive_launch"]


def _pts(n, seed):
    return torch.from_numpy(synth.uniform(n, 3, seed=seed) * np.float32(10.0)).cuda()


def _tiles(X, nu):
    return smx.triplet_packed(X, nu, "lambda", stats=True)[0]


@pytest.mark.parametrize("n", [703, 704, 705, 735, 736, 737, 895, 896, 897, 928, 1025])
def test_sizes(n):
    print(f"packed rows n={n}", flush=True)
    X = _pts(n, n)
    assert torch.equal(smx.triplet_packed(X, 0.7), _tiles(X, 0.7))


@pytest.mark.parametrize("kind", KINDS)
def test_maps(kind):
    X = _pts(710, 1)
    assert torch.equal(smx.triplet_packed(X, 1.3, kind), _tiles(X, 1.3))


@pytest.mark.parametrize("shift", [1, 2, 3, 5, 31, 32])
def test_buffer_offsets(shift):
    n = 709
    m = math.comb(n, 3)
    X = _pts(n, 2)
    buf = torch.full((m + 64,), -7.0, device="cuda")
    smx.triplet_packed(X, 1.0, out=buf[shift:shift + m])
    assert torch.equal(buf[shift:shift + m], _tiles(X, 1.0))
    assert (buf[:shift] == -7.0).all() and (buf[shift + m:] == -7.0).all()


def test_strided_positions():
    X = _pts(720, 3)
    wide = torch.zeros((720, 7), device="cuda")
    wide[:, :3] = X
    assert torch.equal(smx.triplet_packed(wide[:, :3], 1.0), _tiles(X, 1.0))
