"""Axilrod-Teller matrix form where particles are much nearer to each other than to
the rest: bonds (the energy's terms largely cancel) and one very close pair (the
FP16 operands of its rows span many powers of two).

Tolerances.  Bonds: 1e-5, the bar of the FP32 kernels.  One pair at r of the
others' spacing: an entry of its two rows is off by up to 2^-25 at a scale where the
nearest is 2^12, 2^-37 r^-3 of an entry at the spacing; over ten forms of up to
2.8 / r^3, two operands, a cancellation of about 5 in the forms' sum and 25 / 8 for
the slow fall of the far entries' errors that is about 1000 2^-37 r^-3 = 2^-27 r^-3 of
what the pair gets, beside 1e-5.  Neither may be further off than the FP32 triplet
loop, which a workspace of its own size selects, by more than 1e-6.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu

AT = smx.Pot(nu=1.0, at=True, lj=False)


def _loop_ws(n):
    return torch.empty(smx.triplet_workspace_bytes(n, AT, limit=0), dtype=torch.uint8, device="cuda")


def _liquid(n, seed):
    return synth.rsa(n, seed=seed, side=20.0 * (n / 8192) ** (1 / 3), dmin=0.8).astype(np.float64)


def _bonds(n, bond, share, seed):
    """`share` of n particles in pairs at `bond`, centres and the others 0.8 apart, random order."""
    r = np.random.default_rng(seed)
    pairs = int(n * share) // 2
    C = _liquid(n - pairs, seed)
    u = r.standard_normal((pairs, 3))
    X = np.concatenate((C, C[:pairs] + bond * u / np.linalg.norm(u, axis=1, keepdims=True)))
    return X[r.permutation(n)].astype(np.float32)


def _exact(X):
    """Energy and gradient in FP64 from the dipole tensors of all pairs, E = -tr(T^3) / 18."""
    x = torch.from_numpy(X).cuda().double()
    n = x.shape[0]
    T = torch.zeros((n, 3, n, 3), dtype=torch.float64, device="cuda")
    eye = torch.eye(3, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 24) // n)

    def pairs(a, b):
        d = x[a:b, None] - x[None]
        s = d.square().sum(-1)
        s[torch.arange(b - a), torch.arange(a, b)] = float("inf")
        return d, s

    for a in range(0, n, step):
        b = min(n, a + step)
        d, s = pairs(a, b)
        t = 3 * s.pow(-2.5)[..., None, None] * d[..., :, None] * d[..., None, :] - s.pow(-1.5)[..., None, None] * eye
        T[a:b] = t.permute(0, 2, 1, 3)
    T = T.view(3 * n, 3 * n)
    S = (T @ T).view(n, 3, n, 3)
    e = -(T.view(n, 3, n, 3) * S).sum().item() / 18
    G = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    for a in range(0, n, step):
        b = min(n, a + step)
        d, s = pairs(a, b)
        P = S[a:b].permute(0, 2, 1, 3)
        P = P + P.transpose(2, 3)
        q = (P * d[..., None, :]).sum(-1)
        xq, tr, d5 = (d * q).sum(-1) / 2, P.diagonal(dim1=2, dim2=3).sum(-1) / 2, s.pow(-2.5)
        G[a:b] = -((3 * d5)[..., None] * (q + tr[..., None] * d) - (15 * xq * d5 / s)[..., None] * d).sum(1) / 3
    return e, G


def _errors(Xt, e, G, ws):
    """Relative errors of the energy, of both calls, and of the gradient (largest norm)."""
    E1 = smx.triplet_energy(Xt, AT, ws=ws)
    E2, g = smx.triplet_energy_grad(Xt, AT, ws=ws)
    err = (g.double() - G).norm(dim=1).max() / G.norm(dim=1).max()
    return abs(E1[0].item() - e) / abs(e), abs(E2[0].item() - e) / abs(e), err.item()


def test_exact_is_the_oracle():
    X = _bonds(300, 0.3, 1.0, 1)
    e, G = _exact(X)
    assert abs(e - oracle.at_energy(X)) <= 1e-11 * abs(e)
    ref = np.asarray(oracle.at_grad(X))
    assert np.abs(G.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()


# one call below the 256-wide tiles, one where the device turns them down
@pytest.mark.parametrize("n", [2051, 8192])
@pytest.mark.parametrize("bond,share", [(0.3, 1.0), (0.2, 1.0), (0.3, 0.3)])
def test_bonds(n, bond, share):
    X = _bonds(n, bond, share, 10)
    e, G = _exact(X)
    got = _errors(torch.from_numpy(X).cuda(), e, G, None)
    loop = _errors(torch.from_numpy(X).cuda(), e, G, _loop_ws(n))
    print(f"bonds n={n} {bond} x {share}: energy, energy, gradient", ["%.1e" % v for v in got], "loop",
          ["%.1e" % v for v in loop], flush=True)
    for v, v0 in zip(got, loop):
        assert v <= 1e-5
        assert v <= max(v0, 1e-6) * 3  # neither error is more than a few roundings' chance there


@pytest.mark.parametrize("r", [0.3, 0.1, 0.01, 0.003])
@pytest.mark.parametrize("n", [1100, 4200])
def test_one_close_pair(n, r):
    X = _liquid(n, 7)
    u = np.array([0.48, -0.6, 0.64])
    X[n // 2] = X[n // 3].astype(np.float32) + r * u
    X = X.astype(np.float32)
    e, G = _exact(X)
    got = _errors(torch.from_numpy(X).cuda(), e, G, None)
    loop = _errors(torch.from_numpy(X).cuda(), e, G, _loop_ws(n))
    print(f"pair n={n} at {r}:", ["%.1e" % v for v in got], "loop", ["%.1e" % v for v in loop], flush=True)
    for v, v0 in zip(got, loop):
        assert v <= 1e-5 + 2.0 ** -27 * r ** -3
        assert v <= max(v0, 1e-6)


@pytest.mark.parametrize("kind", ["lambda", "bbox", "linear", "lambda_below", "recursive", "recursive_launch"])
def test_either_tile_on_every_map(kind):
    """Liquid (256-wide tiles) and bonds (128-wide), n past both, against the plain order."""
    n = 4200
    for X in (_liquid(n, 3).astype(np.float32), _bonds(n, 0.3, 1.0, 3)):
        Xt = torch.from_numpy(X).cuda()
        E0, G0 = smx.triplet_energy_grad(Xt, AT, "linear")
        E, G = smx.triplet_energy_grad(Xt, AT, kind)
        assert abs(E[0].item() - E0[0].item()) <= 1e-5 * abs(E0[0].item())
        assert (G - G0).norm(dim=1).max() <= 1e-6 * G0.norm(dim=1).max()
