"""4-point contacts without statistics: the lists of work items and the gate that
sends a graph to the 4-simplex tiles once counting from its contacts costs more.
The cost is the number of pairs of forward contacts, sum_i C(f_i, 2), its limit
max(4.5e6, n^3 / 6000) (n^3 / 3200 past 8192).  Counts are exact, against the oracle or the count of the
calls with statistics (always the tiles, ungated)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu


def _even(n, seed):
    return synth.uniform(n, 3, seed=seed) * np.float32(n ** (1 / 3))


def _cluster(n, m, consecutive, seed):
    """m of n even particles, moved to where all of them are in contact (rc >= 1)."""
    X = _even(n, seed)
    r = np.random.default_rng(seed)
    ids = 100 + np.arange(m) if consecutive else np.sort(r.permutation(n)[:m])
    X[ids] = (r.random((m, 3)) * 0.3 - 50.0).astype(np.float32)
    return X


def _cost(X, rc):
    f = np.zeros(len(X), np.int64)
    rc2 = np.float32(rc * rc)
    for i in range(len(X) - 1):
        d = X[i + 1:] - X[i]
        f[i] = int(((d * d).sum(1) < rc2).sum())
    return int((f * (f - 1) // 2).sum())


def _count(X, rc, kind="lambda", **kw):
    return int(smx.quad_contacts(torch.from_numpy(X).cuda(), rc, kind, **kw).item())


def _tiles(X, rc):
    c, s = smx.quad_contacts(torch.from_numpy(X).cuda(), rc, stats=True)
    assert int(s[0]) == math.comb(len(X), 4)
    return int(c.item())


# just under and over the limit, where the tiles' ids need more than one round of the
# gated launch (nb > 64), and at sizes with one, two and four words a lane
@pytest.mark.parametrize("n,rc,dense", [(1100, 3.6, False), (1100, 4.2, True), (4200, 2.9, False), (4200, 3.9, True),
                                        (8200, 2.0, False), (9000, 6.0, True)])
def test_either_side_of_the_gate(n, rc, dense):
    X = _even(n, 21)
    assert (_cost(X, rc) > max(4500000, n ** 3 // (6000 if n <= 8192 else 3200))) == dense
    ref = _tiles(X, rc)
    assert ref > 0
    for kind in ("lambda", "linear", "recursive") if n < 9000 else ("lambda",):
        print(f"gate n={n} rc={rc} {kind}", flush=True)
        assert _count(X, rc, kind) == ref


@pytest.mark.parametrize("kind", ["bbox", "recursive_launch"])
def test_dense_on_the_other_maps(kind):
    X = _even(1100, 22)
    assert _cost(X, 4.2) > 4500000
    assert _count(X, 4.2, kind) == oracle.quad_contacts(X, 4.2)


# clusters fill whole words and tiles (items by rows, then by columns; lists past their end)
@pytest.mark.parametrize("n,m,consecutive", [(256, 100, True), (1000, 130, True), (1000, 400, False), (1100, 200, True),
                                             (1500, 300, True), (1500, 1500, True), (3000, 150, True), (3000, 300, False),
                                             (4200, 65, True), (8200, 150, True)])
def test_clusters(n, m, consecutive):
    X = _cluster(n, m, consecutive, n + m) if m < n else _even(n, 3) * np.float32(0.01)
    ref = math.comb(n, 4) if m == n else _tiles(X, 1.3)
    assert ref >= math.comb(m, 4)
    print(f"cluster n={n} m={m}", flush=True)
    assert _count(X, 1.3) == ref


def test_workspace_without_the_lists():
    """A workspace of the tile form's size is enough for any call."""
    n = 2100
    X = _even(n, 5)
    nb = -(-n // 64)
    least = (65536 + 512 * nb * nb + 255) // 256 * 256
    assert least < smx.workspace_bytes(3, n)
    ref = oracle.quad_contacts(X, 2.0)
    for size in (least, smx.workspace_bytes(3, n) - 1, smx.workspace_bytes(3, n)):
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
        assert _count(X, 2.0, ws=ws) == ref
    with pytest.raises(ValueError):
        smx.quad_contacts(torch.from_numpy(X).cuda(), 2.0, ws=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))


def test_calls_share_nothing():
    """Dense, sparse, dense in turn through one workspace, and on two streams."""
    n = 2100
    X = torch.from_numpy(_even(n, 6)).cuda()
    dense, sparse = (int(smx.quad_contacts(X, rc, stats=True)[0].item()) for rc in (4.5, 1.6))
    ws = torch.empty(smx.workspace_bytes(3, n), dtype=torch.uint8, device="cuda")
    for rc, ref in ((4.5, dense), (1.6, sparse)) * 3:
        assert int(smx.quad_contacts(X, rc, ws=ws).item()) == ref
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = []
    for k in range(6):
        with torch.cuda.stream(streams[k % 2]):
            got.append((smx.quad_contacts(X, (4.5, 1.6)[k % 2]), (dense, sparse)[k % 2]))
    torch.cuda.synchronize()
    assert all(int(g.item()) == ref for g, ref in got)


@pytest.mark.parametrize("m,consecutive", [(300, True), (700, True), (1400, True), (1400, False)])
def test_a_cluster_is_no_slower_than_the_tiles(m, consecutive):
    """The calls with statistics take the tiles (and count them beside)."""
    X = torch.from_numpy(_cluster(8192, m, consecutive, 7)).cuda()
    ws = torch.empty(smx.workspace_bytes(3, 8192), dtype=torch.uint8, device="cuda")

    def best(stats):
        ts = []
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            smx.quad_contacts(X, 1.3, stats=stats, ws=ws)
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b))
        return min(ts)

    t, t0 = best(False), best(True)
    print(f"cluster of {m}: {t:.2f} ms, tiles with statistics {t0:.2f} ms", flush=True)
    assert t <= 1.2 * t0
