"""Device memory that the binding takes for itself: no more than a call can use,
and less where the device has no room for it."""
import math

import numpy as np
import pytest
import torch

import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu


def _particles(n, seed=1):
    return torch.from_numpy(synth.rsa(n, seed=seed, side=20.0 * (n / 8192) ** (1 / 3), dmin=0.8)).cuda()


def _peak(f):
    """Bytes a call allocates beside what is there."""
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    out = f()
    torch.cuda.synchronize()
    return torch.cuda.max_memory_allocated() - before, out


def test_calls_without_matrix_products_take_little():
    X = torch.from_numpy(synth.uniform(20000, 3, seed=1) * np.float32(27.0)).cuda()
    lj = smx.Pot(at=False, lj=True, rc=0.9)
    few = 4 << 20
    assert _peak(lambda: smx.triplet_energy(X, lj))[0] < few
    assert _peak(lambda: smx.triplet_energy_grad(X, lj))[0] < few
    assert _peak(lambda: smx.triplet_energy_backward(X, torch.ones((), device="cuda"), lj))[0] < few
    P = _particles(2000)
    assert _peak(lambda: smx.triplet_energy(P, smx.Pot(), stats=True))[0] < few
    assert _peak(lambda: smx.triplet_energy(P[:900], smx.Pot()))[0] < few
    D = torch.empty(6000 * 6001 // 2, device="cuda")
    Z = torch.from_numpy(synth.normal(6000, 35, seed=2)).cuda()
    assert _peak(lambda: smx.edm_packed(Z, out=D))[0] == 0


@pytest.fixture
def cap():
    """Leaves the allocator `extra` bytes beside what it has handed out."""
    total = torch.cuda.get_device_properties(0).total_memory

    def set_cap(extra):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + extra) / total)

    yield set_cap
    torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("room", [1 << 30, 300 << 20, 64 << 20, 8 << 20])
def test_triplets_in_little_memory(cap, room):
    """Fewer forms at a time, fewer columns, the triplet loop: the same results to
    FP32 accuracy (1e-5 of the largest force, as against the oracle)."""
    n = 4096
    X = _particles(n).requires_grad_(True)
    E0, G0 = smx.triplet_energy_grad(X.detach())
    need = smx.triplet_workspace_bytes(n)
    assert need > 600 << 20
    cap(room)
    print(f"room {room >> 20} MB of {need >> 20}", flush=True)
    peak, e = _peak(lambda: smx.TripletEnergy.apply(X))
    assert peak <= room
    e.backward()
    assert abs(e.item() - E0[0].item()) <= 1e-5 * abs(E0[0].item())
    assert (X.grad - G0).norm(dim=1).max() <= 1e-5 * G0.norm(dim=1).max()
    E1 = smx.triplet_energy(X.detach())
    assert abs(E1[0].item() - E0[0].item()) <= 1e-5 * abs(E0[0].item())


def test_distances_in_little_memory(cap):
    n, d = 8192, 600
    X = torch.from_numpy(synth.normal(n, d, seed=3)).cuda()
    D = torch.empty(n * (n + 1) // 2, device="cuda")
    ref = smx.edm_packed(X, out=D, ws=torch.empty(32768, dtype=torch.uint8, device="cuda")).clone()
    for stats in (True, False):
        D.zero_()
        cap(4 << 20)
        got = smx.edm_packed(X, out=D, stats=stats)
        torch.cuda.set_per_process_memory_fraction(1.0)  # the comparison takes memory too
        assert torch.equal(D, ref)
        assert not stats or int(got[1][0]) == n * (n + 1) // 2


@pytest.mark.parametrize("shift", [4, 8, 24])
def test_unaligned_workspaces(shift):
    """FP32 distances accept any alignment that the statistics slots allow (none
    without them) and then take the difference form; triplets align their operands."""
    n, d = 8192, 40
    X = torch.from_numpy(synth.normal(n, d, seed=4)).cuda()
    ref = smx.edm_packed(X, ws=torch.empty(32768, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(smx.workspace_bytes(1, n, d) + 64, dtype=torch.uint8, device="cuda")[shift:]
    assert torch.equal(smx.edm_packed(X, ws=ws), ref)
    if shift % 8 == 0:
        got, st = smx.edm_packed(X, ws=ws, stats=True)
        assert torch.equal(got, ref) and int(st[0]) == n * (n + 1) // 2
        P = _particles(1100)
        E0, G0 = smx.triplet_energy_grad(P)
        ws = torch.empty(smx.workspace_bytes(2, 1100) + 64, dtype=torch.uint8, device="cuda")[shift:]
        E, G = smx.triplet_energy_grad(P, ws=ws)
        assert abs(E[0].item() - E0[0].item()) <= 1e-5 * abs(E0[0].item())
        assert (G - G0).norm(dim=1).max() <= 1e-5 * G0.norm(dim=1).max()
