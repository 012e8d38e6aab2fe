"""FP32 distances on the matrix cores (n >= 8192 with d >= 36, n >= 5120 with d >=
65, given the workspace): every pair to FP32 accuracy, the difference form being
the other path (a workspace of 32768 bytes selects it).

Tolerance: |D^ - D| / D <= 1e-5 as for the difference form.  A kept Gram value is
at least 5/16 of |x_i|^2 + |x_j|^2, so its few roundings at that size are at most
about 16/5 * 4 * 2^-24 = 8e-7 of D; every other pair is a sum of squares.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

KINDS = ["lambda", "bbox", "linear", "lambda_below", "recursive", "recursive_launch"]


def _diff(X, kind="lambda"):
    return smx.edm_packed(X, kind, ws=torch.empty(32768, dtype=torch.uint8, device="cuda"))


def _row(n, i):
    return i * n - i * (i - 1) // 2


def _check_rows(D, X, rows):
    n = X.shape[0]
    for i in rows:
        got = D[_row(n, i):_row(n, i) + n - i].cpu().numpy().astype(np.float64)
        ref = oracle.edm_rows(X, i, i + 1)
        assert got[0] == 0.0
        far = ref > 0
        assert (got[~far] == 0.0).all()
        if far.any():
            assert np.max(np.abs(got[far] - ref[far]) / ref[far]) <= 1e-5


def _data(kind, n, d, seed):
    X = synth.normal(n, d, seed=seed)
    r = np.random.default_rng(seed)
    if kind == "offset":
        X = X * np.float32(0.1) + np.float32(50.0)
    elif kind == "clusters":
        X = (X * np.float32(0.01) + r.standard_normal((8, d)).astype(np.float32)[r.integers(0, 8, n)])
    elif kind == "few_near":
        X[n - 40:] = X[:40] + np.float32(1e-3)
        X[200] = X[201]
    elif kind == "block_near":  # whole tiles of near pairs, in few of the samples
        X[1024:1280] = X[1024] + np.float32(1e-2) * X[1024:1280]
    return np.ascontiguousarray(X.astype(np.float32))


# first sizes, tile edges, one row past a tile; d at the ends of a k block
@pytest.mark.parametrize("n,d", [(5119, 65), (5120, 65), (5121, 66), (6000, 64), (8191, 37), (8192, 36), (8193, 37), (8320, 48), (8325, 100)])
def test_sizes_and_maps(n, d):
    print(f"edm matrix n={n} d={d}", flush=True)
    X = _data("few_near", n, d, seed=n + d)
    Xt = torch.from_numpy(X).cuda()
    D = smx.edm_packed(Xt)
    _check_rows(D, X, [0, 1, 95, 127, 128, 200, 1023, n - 130, n - 129, n - 40, n - 2, n - 1])
    for kind in KINDS[1:]:
        assert torch.equal(D, smx.edm_packed(Xt, kind)), kind
    rel = ((D - _diff(Xt)).abs() / D.clamp_min(1e-30)).max().item()
    assert rel <= 2e-5


@pytest.mark.parametrize("kind", ["normal", "offset", "clusters", "few_near", "block_near"])
def test_inputs(kind):
    n, d = 8260, 40
    X = _data(kind, n, d, seed=5)
    D = smx.edm_packed(torch.from_numpy(X).cuda())
    _check_rows(D, X, [0, 17, 128, 200, 1024, 1100, 4096, 8200, n - 1])


@pytest.mark.parametrize("kind", ["few_near", "block_near", "clusters"])
def test_tiled_layout_and_statistics_hold_the_same_values(kind):
    n, d = 8200, 36
    Xt = torch.from_numpy(_data(kind, n, d, seed=2)).cuda()
    D = smx.edm_packed(Xt)
    S, st = smx.edm_packed(Xt, stats=True)
    assert torch.equal(D, S) and int(st[0]) == n * (n + 1) // 2
    T = smx.edm_tiled(Xt)
    for i in (0, 100, 127, 128, 1030, n - 300, n - 1):
        j = torch.arange(i, n, device="cuda")
        off = ((j // 128) * (j // 128 + 1) // 2 + i // 128) * 16384 + (i % 128) * 128 + j % 128
        assert torch.equal(T[off], D[_row(n, i):_row(n, i) + n - i])


def test_not_finite_as_the_difference_form():
    n, d = 8195, 36
    X = _data("normal", n, d, seed=8)
    X[3, 5], X[700, 2], X[900, 2], X[1100, 7] = np.nan, np.inf, np.inf, -np.inf
    X[2000] *= np.float32(1e25)
    Xt = torch.from_numpy(X).cuda()
    D, R = smx.edm_packed(Xt), _diff(Xt)
    assert torch.equal(torch.isnan(D), torch.isnan(R)) and torch.equal(torch.isinf(D), torch.isinf(R))
    fine = torch.isfinite(R) & (R > 0)
    assert ((D[fine] - R[fine]).abs() / R[fine]).max().item() <= 2e-5


@pytest.mark.parametrize("shift", [1, 7, 32])
def test_buffers_and_strides(shift):
    n, d = 8193, 36
    X = _data("few_near", n, d, seed=9)
    wide = torch.zeros((n, d + 5), device="cuda")
    wide[:, :d] = torch.from_numpy(X)
    m = n * (n + 1) // 2
    buf = torch.full((m + 64,), -7.0, device="cuda")
    smx.edm_packed(wide[:, :d], out=buf[shift:shift + m])
    assert torch.equal(buf[shift:shift + m], smx.edm_packed(torch.from_numpy(X).cuda()))
    assert (buf[:shift] == -7.0).all() and (buf[shift + m:] == -7.0).all()
