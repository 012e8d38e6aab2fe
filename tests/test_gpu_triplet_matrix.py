"""GPU parity of the Axilrod-Teller matrix form (n >= 768) at the edges of its
pair tiles, of its column chunks and of the plans that a smaller workspace
allows, against the FP64 oracle.

Tolerances: energy |E^ - E| <= 1e-5 |E| and gradient max_i |G^_i - G_i| <= 1e-5
max_i |G_i|, the bars of the FP32 kernels.  The matrix form holds its operands to
2^-23 and accumulates in FP32 over at most 3 n / 16 steps, so its error is of the
order of sqrt(3 n / 16) 2^-24, 3e-6 at n = 8192.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

AT = smx.Pot(nu=0.8, at=True, lj=False)
KINDS = ["lambda", "bbox", "linear", "lambda_below", "recursive", "recursive_launch"]
BASE = 3 * 256 * 128  # the loop form's workspace: slots, then 24 bytes a particle


def _pts(n, seed):
    return synth.rsa(n, seed=seed, side=20.0 * (n / 8192) ** (1 / 3), dmin=0.8)


def _check(X, kind="lambda", ws=None, rows=None):
    n = X.shape[0]
    print(f"matrix form n={n} {kind} ws={None if ws is None else ws.numel()}", flush=True)
    Xt = torch.from_numpy(X).cuda()
    e_ref = 0.8 * oracle.at_energy(X)
    E = smx.triplet_energy(Xt, AT, kind, ws=ws)
    E2, G = smx.triplet_energy_grad(Xt, AT, kind, ws=ws)
    torch.cuda.synchronize()
    for e in (E[0].item(), E2[0].item(), E2[1].item()):
        assert abs(e - e_ref) <= 1e-5 * abs(e_ref)
    g = G.cpu().numpy().astype(np.float64)
    if rows is None:
        rows = np.arange(n)
        ref = 0.8 * oracle.at_grad(X)
    else:
        rows = np.asarray(rows)
        ref = 0.8 * np.asarray(oracle.at_grad_rows(X, rows))
    err = np.linalg.norm(g[rows] - ref, axis=1).max() / np.linalg.norm(g, axis=1).max()
    print(f"  energy {abs(E2[0].item() - e_ref) / abs(e_ref):.1e} gradient {err:.1e}", flush=True)
    assert err <= 1e-5
    return g


# below, at and past a tile (128) and a k block (32); the first sizes of both calls
@pytest.mark.parametrize("n", [767, 768, 769, 895, 1023, 1024, 1025, 1057])
def test_sizes(n):
    _check(_pts(n, seed=n), rows=[0, 1, 127, 128, 255, 256, 511, 640, n - 130, n - 2, n - 1])


@pytest.mark.parametrize("kind", KINDS)
def test_maps(kind):
    n = 1030
    _check(_pts(n, seed=5), kind, rows=[0, 127, 128, 500, n - 7, n - 1])


@pytest.mark.parametrize("n", [4095, 4097])
def test_tile_256(n):
    """Both sides of the switch to 256-wide tiles, last tile ragged or one row."""
    rows = [0, 255, 256, 2047, 2048, n - 257, n - 2, n - 1]
    X = _pts(n, seed=n)
    g = _check(X, rows=rows)
    # every row against the triplet loop (which a workspace of its own size selects)
    ws = torch.empty(BASE + 24 * n + 256, dtype=torch.uint8, device="cuda")
    _, L = smx.triplet_energy_grad(torch.from_numpy(X).cuda(), AT, ws=ws)
    L = L.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(g - L, axis=1).max() <= 2e-5 * np.linalg.norm(L, axis=1).max()


@pytest.mark.parametrize("room", ["five", "two", "one", "columns"])
def test_plans(room):
    """Workspaces that hold five, two or one form at a time, or 2048 columns of one."""
    n = 2309
    rows32, cols32 = -(-n // 32) * 32, -(-n // 32) * 32
    panel = 4 * rows32 * (2048 if room == "columns" else cols32)
    forms = {"five": 5, "two": 2, "one": 1, "columns": 1}[room]
    head = (BASE + 24 * n + 255) // 256 * 256 + (4 * n + 255) // 256 * 256 + 256
    ws = torch.empty(head + forms * panel, dtype=torch.uint8, device="cuda")
    _check(_pts(n, seed=3), ws=ws, rows=[0, 127, 128, 1151, 2047, 2048, n - 6, n - 1])


def test_wide_rows_and_scale():
    """Positions in a strided matrix, and the same cluster in units 1000 times
    smaller and larger: the energy scales by the ninth power."""
    X = _pts(800, seed=9)
    wide = torch.zeros((800, 5), device="cuda")
    wide[:, :3] = torch.from_numpy(X)
    e0 = smx.triplet_energy_grad(wide[:, :3], AT)[0][0].item()
    assert abs(e0 - 0.8 * oracle.at_energy(X)) <= 1e-5 * abs(e0)
    for f in (1.0 / 1024, 1024.0):
        e = smx.triplet_energy_grad(wide[:, :3] * f, AT)[0][0].item()
        assert abs(e * f ** 9 - e0) <= 1e-6 * abs(e0)


def test_coincident_pair_is_not_finite():
    X = _pts(900, seed=2)
    X[7] = X[411]
    E, G = smx.triplet_energy_grad(torch.from_numpy(X).cuda(), AT)
    assert not torch.isfinite(E[0]).item() and not torch.isfinite(G[7]).any().item()
