"""The work this library is used for, as timed cases: packed distance matrices,
Axilrod-Teller (+ Lennard-Jones) energies and gradients, per-triplet energies,
4-point contact counts, the cellular automaton on the triangle of cells and the
map dump, each through the binding's public calls.

Particles are liquid-like as the library's own sets: about one per unit volume
and none closer than 0.8, in random order.  Points of the distance matrices are
N(0, 1), cells are alive with probability 0.3.

Energies come back from the library in double precision because they are summed
in it; the programs here join them to the rest of an FP32 model and hold them in
the type of the positions.
"""
from __future__ import annotations

import math

import torch

import paper_1610_07394_amd as smx

DEV = "cuda"


def listed():
    return [
        # the small distance matrix of the library's examples (n = 1024 points in space): a call
        # of a few microseconds, where latency and launches count
        {"name": "edm_fp32_small", "path": "edm", "n": 1024, "d": 3, "prec": "fp32", "map": "lambda", "pad": 0},
        # an ordinary feature set of odd sizes (no multiple of a tile, rows not 16-byte aligned)
        {"name": "edm_fp32_ragged", "path": "edm", "n": 9001, "d": 37, "prec": "fp32", "map": "lambda", "pad": 0},
        # the benchmark's full-size distance matrix, 8.6 GB of output
        {"name": "edm_fp32_large", "path": "edm", "n": 65536, "d": 64, "prec": "fp32", "map": "lambda", "pad": 0},
        # BF16 Gram form at the ragged size of the tests (last tile partly filled, k padded)
        {"name": "edm_bf16_ragged", "path": "edm", "n": 16484, "d": 300, "prec": "bf16", "map": "lambda", "pad": 0},
        # split-BF16 Gram form of the benchmark: embeddings of 512 dimensions
        {"name": "edm_split_large", "path": "edm", "n": 32768, "d": 512, "prec": "split_bf16", "map": "lambda",
         "pad": 0},
        # forces on a small cluster: the inner call of a molecular-dynamics or relaxation loop
        {"name": "at_lj_grad_small", "path": "forces", "n": 500, "lj": True, "map": "lambda"},
        # energy of one configuration (Monte Carlo, screening): forward alone, odd size
        {"name": "at_energy", "path": "energy", "n": 2051, "lj": False, "map": "lambda"},
        # the benchmark's training step: Axilrod-Teller + Lennard-Jones energy forward and backward
        {"name": "at_lj_step_large", "path": "step", "n": 8192, "lj": True, "fused": True, "map": "lambda"},
        # one energy per triplet in packed order, 5.7 GB of output: features of all triplets
        {"name": "triplet_packed", "path": "packed", "n": 2048, "map": "lambda"},
        # 4-point correlation count of the benchmark's particles
        {"name": "quad_contacts", "path": "quad", "n": 8192, "rc": 2.0, "map": "lambda"},
        # one generation of the automaton at the benchmark's size
        {"name": "life_large", "path": "life", "n": 32768, "map": "lambda"},
        # the block-space map itself over the 3-simplex: tiles, element counts and checksum
        {"name": "map3_dump", "path": "map", "m": 3, "n": 1024, "rho": 8, "strict": True, "map": "lambda"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the paths in about the shares they have above, every map
    now and then, sizes log-uniform from a handful of tiles to the largest."""
    path = rng.choice(["edm", "edm", "edm", "edm", "forces", "energy", "step", "step", "packed", "quad", "life",
                       "map"])
    kind = rng.choice(["lambda", "lambda", "lambda", "lambda", "bbox", "linear"])
    if path == "edm":
        prec = rng.choice(["fp32", "fp32", "bf16", "split_bf16"])
        d = _log(rng, 2, 200) if prec == "fp32" else _log(rng, 16, 600)
        n = _log(rng, 300, 40000 if d <= 64 else 20000)
        return {"path": path, "n": n, "d": d, "prec": prec, "map": kind, "pad": rng.choice([0, 0, 0, 1, 4])}
    if path in ("forces", "energy", "step"):
        c = {"path": path, "n": _log(rng, 100, 7000), "lj": rng.random() < 0.5, "map": kind}
        if path == "step":
            c["fused"] = rng.random() < 0.7
        return c
    if path == "packed":
        return {"path": path, "n": _log(rng, 60, 2000), "map": kind}
    if path == "quad":
        return {"path": path, "n": _log(rng, 300, 8000), "rc": round(rng.uniform(1.1, 2.6), 3), "map": kind}
    if path == "life":
        return {"path": path, "n": _log(rng, 500, 32000), "map": kind}
    m = rng.choice([2, 3])
    rho = rng.choice([8, 16, 32]) if m == 2 else rng.choice([4, 8, 16])
    n = _log(rng, 500, 16000) if m == 2 else _log(rng, 100, 1000)
    return {"path": path, "m": m, "n": n, "rho": rho, "strict": rng.random() < 0.5, "map": kind}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _particles(n, seed):
    """n particles at the density of 8192 in a cube of side 20, on random sites
    of a cubic lattice, each moved by as much as keeps every pair 0.8 apart."""
    g = _gen(seed)
    m = 1
    while m ** 3 < n:
        m += 1
    a = max(20.0 * (n / 8192) ** (1 / 3) / m, 0.85)
    site = torch.randperm(m ** 3, generator=g, device=DEV)[:n]
    xyz = torch.stack((site % m, site // m % m, site // (m * m)), 1).double()
    move = (torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64) - 0.5) * (a - 0.8)
    return (xyz * a + move).float().contiguous()


def _pot(case):
    return smx.Pot(nu=1.0, at=True, lj=bool(case.get("lj", False)), eps=1.0, sigma=1.0, rc=3.0)


def prepare(case, seed):
    c = dict(case)
    path = c["path"]
    if path == "edm":
        wide = torch.randn((c["n"], c["d"] + c["pad"]), generator=_gen(seed), device=DEV, dtype=torch.float32)
        s = {"X": wide[:, : c["d"]]}
        if c["n"] >= 4096:  # a program with a large matrix keeps its buffer
            s["D"] = torch.empty(c["n"] * (c["n"] + 1) // 2, dtype=torch.float32, device=DEV)
        return {"case": c, **s}
    if path in ("forces", "energy", "quad"):
        return {"case": c, "X": _particles(c["n"], seed), "pot": _pot(c)}
    if path == "step":
        return {"case": c, "X": _particles(c["n"], seed).requires_grad_(True), "pot": _pot(c)}
    if path == "packed":
        return {"case": c, "X": _particles(c["n"], seed),
                "E": torch.empty(math.comb(c["n"], 3), dtype=torch.float32, device=DEV)}
    if path == "life":
        cells = torch.rand(smx.life_len(c["n"]), generator=_gen(seed), device=DEV) < 0.3
        cells = cells.to(torch.uint8)
        return {"case": c, "S": cells, "D": torch.empty_like(cells)}
    # the map has no input data; the seed moves n within the last tile
    c["n"] -= seed % c["rho"]
    return {"case": c}


# ------------------------------------------------------------------ one pass
def run(state):
    c = state["case"]
    path = c["path"]
    if path == "edm":
        return smx.edm_packed(state["X"], c["map"], c["prec"], out=state.get("D"))
    if path == "forces":
        E, G = smx.triplet_energy_grad(state["X"], state["pot"], c["map"])
        return {"E": E.to(G.dtype), "G": G}
    if path == "energy":
        return smx.triplet_energy(state["X"], state["pot"], c["map"]).to(state["X"].dtype)
    if path == "step":
        X = state["X"]
        X.grad = None
        loss = smx.TripletEnergy.apply(X, state["pot"], c["map"], c["fused"]).to(X.dtype)
        loss.backward()
        return {"loss": loss.detach(), "grad": X.grad}
    if path == "packed":
        return smx.triplet_packed(state["X"], 1.0, c["map"], out=state["E"])
    if path == "quad":
        return smx.quad_contacts(state["X"], c["rc"], c["map"])
    if path == "life":
        return smx.simplex_life(state["S"], c["n"], c["map"], out=state["D"])
    dump = smx.simplex_map2 if c["m"] == 2 else smx.simplex_map3
    tiles, stats = dump(c["n"], c["rho"], c["map"], strict=c["strict"], tiles=True, stats=True)
    return {"tiles": tiles, "stats": stats}


def work(case):
    n, path = case["n"], case["path"]
    pairs, tri = n * (n + 1) // 2, math.comb(n, 3)
    if path == "edm":
        d, terms = case["d"], {"fp32": 3, "bf16": 2, "split_bf16": 6}[case["prec"]]
        return {"bytes": 4 * n * d + 4 * pairs, "flops": terms * d * pairs}
    if path == "energy":
        return {"bytes": 12 * n, "flops": 20 * tri}
    if path in ("forces", "step"):
        return {"bytes": 24 * n, "flops": 80 * tri}
    if path == "packed":
        return {"bytes": 12 * n + 4 * tri, "flops": 21 * tri}
    if path == "quad":  # the contact graph: one squared distance per pair, then its 4-cliques
        return {"bytes": 12 * n, "flops": 8 * pairs}
    if path == "life":
        return {"bytes": 2 * smx.life_len(n), "flops": 0}
    nb = -(-n // case["rho"])
    tiles = nb * (nb + 1) // 2 if case["m"] == 2 else nb * (nb + 1) * (nb + 2) // 6
    elems = pairs if case["m"] == 2 else n * (n + 1) * (n + 2) // 6
    return {"bytes": 4 * case["m"] * tiles, "flops": 10 * elems}


# ------------------------------------------------------------------ 64 bits
def _exact_edm(X, n, d):
    """sum_k (x_ik - x_jk)^2 over the packed upper triangle, rows in chunks."""
    Xt = X.double().t().contiguous()
    out = torch.empty(n * (n + 1) // 2, dtype=torch.float64, device=DEV)
    step = max(1, min(n, (1 << 26) // n))
    for a in range(0, n, step):
        b = min(n, a + step)
        acc = torch.zeros((b - a, n - a), dtype=torch.float64, device=DEV)
        for k in range(d):
            acc += (Xt[k, a:b, None] - Xt[k, None, a:]).square_()
        keep = torch.arange(n - a, device=DEV)[None] >= torch.arange(b - a, device=DEV)[:, None]
        at = a * n - a * (a - 1) // 2
        got = acc[keep]
        out[at:at + got.numel()] = got
    return out


def _exact_at(X, lj):
    """Energy (total, Axilrod-Teller, Lennard-Jones) and gradient.

    With the dipole tensors T_ij = 3 x x^T / r^5 - 1 / r^3 of the pairs, a
    triplet's (1 + 3 cos cos cos) / (r r r)^3 is -tr(T_ij T_jk T_ki) / 3, so over
    all triplets E = -tr(T^3) / 18 with the 3n x 3n matrix of all tensors.
    """
    n = X.shape[0]
    x = X.double()
    T = torch.zeros((n, 3, n, 3), dtype=torch.float64, device=DEV)
    eye = torch.eye(3, dtype=torch.float64, device=DEV)
    step = max(1, min(n, (1 << 24) // n))

    def pairs(a, b):
        dx = x[a:b, None] - x[None]
        s = dx.square().sum(-1)
        s[torch.arange(b - a), torch.arange(a, b)] = math.inf
        return dx, s

    for a in range(0, n, step):
        b = min(n, a + step)
        dx, s = pairs(a, b)
        t = 3 * s.pow(-2.5)[..., None, None] * dx[..., :, None] * dx[..., None, :] - s.pow(-1.5)[..., None, None] * eye
        T[a:b] = t.permute(0, 2, 1, 3)
    T = T.view(3 * n, 3 * n)
    S = (T @ T).view(n, 3, n, 3)
    e_at = -(T.view(n, 3, n, 3) * S).sum() / 18
    G = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    e_lj = torch.zeros((), dtype=torch.float64, device=DEV)
    for a in range(0, n, step):
        b = min(n, a + step)
        dx, s = pairs(a, b)
        Sp = S[a:b].permute(0, 2, 1, 3)
        q = (Sp + Sp.transpose(2, 3)) @ dx[..., None]
        q = q[..., 0]
        xq = (dx * q).sum(-1) / 2
        tr = Sp.diagonal(dim1=2, dim2=3).sum(-1)
        d5 = s.pow(-2.5)
        G[a:b] = -((3 * d5)[..., None] * (q + tr[..., None] * dx) - (15 * xq * d5 / s)[..., None] * dx).sum(1) / 3
        if lj:
            u = torch.where(s < 9.0, 1 / s, torch.zeros_like(s))
            u3 = u ** 3
            e_lj += 2 * (u3 * u3 - u3).sum()
            G[a:b] += (2 * 4 * ((3 * u3 - 6 * u3 * u3) * u)[..., None] * dx).sum(1)
    return e_at + e_lj, e_at, e_lj, G


def _exact_packed(X):
    """(1 + 3 cos cos cos) / (r r r)^3 of every i < j < k, in that order."""
    n = X.shape[0]
    x = X.double()
    out = torch.empty(math.comb(n, 3), dtype=torch.float64, device=DEV)
    at = 0
    for i in range(n - 2):
        v = x[i + 1:] - x[i]
        r = v.square().sum(-1).sqrt()
        b = v[None, :] - v[:, None]  # x_k - x_j
        rb = b.square().sum(-1).sqrt()
        ci = (v @ v.t()) / (r[:, None] * r[None])
        cj = -(b * v[:, None]).sum(-1) / (rb * r[:, None])
        ck = (b * v[None]).sum(-1) / (rb * r[None])
        e = (1 + 3 * ci * cj * ck) / (r[:, None] * r[None] * rb) ** 3
        m = v.shape[0]
        e = e[torch.ones((m, m), dtype=torch.bool, device=DEV).triu_(1)]
        out[at:at + e.numel()] = e
        at += e.numel()
    return out


def exact(case, seed):
    path = case["path"]
    if path in ("quad", "life", "map"):  # whole numbers
        return None
    s = prepare({**case, "n": case["n"]}, seed)
    X = s["X"].detach()
    if path == "edm":
        s.clear()
        return _exact_edm(X, case["n"], case["d"])
    if path == "packed":
        s.clear()
        return _exact_packed(X)
    e, e_at, e_lj, G = _exact_at(X, case["lj"])
    if path == "forces":
        return {"E": torch.stack((e, e_at, e_lj)), "G": G}
    if path == "energy":
        return torch.stack((e, e_at, e_lj))
    return {"loss": e, "grad": G}
