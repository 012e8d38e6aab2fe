"""FP32 distances in many dimensions (d > 512: the preparation reads its rows twice;
d > 8192: the difference form), against the FP64 oracle.

Bar |D^ - D| / D <= 1e-5, as for fewer dimensions.  A kept Gram value is at least 5/16 of
|x_i|^2 + |x_j|^2.  Its operands' own error (2^-23 each, and lo lo^T left out) and the
last two sums are 16/5 * 6 * 2^-24 = 1.2e-6 of D at most; the FP32 sum over 3 d / 8
steps adds up to 3 d / 16 * 2^-24 of it if every rounding falls the same way (9e-5 at d =
8192), its square root, 4e-7 there, otherwise.  The difference form's 2 d roundings in
sequence add more, so the matrix form must not be further off than it either, in the
2-norm, beyond a tenth.

Near pairs are summed as the difference form sums them: equal differences in all of
8191 coordinates round the same way at each step (4e-5 of D), so an element that is
past the bar there has to be the difference form's own, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1610_07394_amd as smx
import synth

pytestmark = pytest.mark.gpu


def _row(D, n, i):
    at = i * n - i * (i - 1) // 2
    return D[at:at + n - i].cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("d", [511, 512, 513, 1000, 2000, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["normal", "offset", "scaled", "near"])
def test_many_dimensions(kind, d):
    n = 5121
    print(f"deep edm {kind} d={d}", flush=True)
    X = synth.normal(n, d, seed=d)
    if kind == "offset":
        X = X * np.float32(0.1) + np.float32(30.0)
    elif kind == "scaled":  # a few coordinates above the others
        X[:, ::97] *= np.float32(30.0)
    elif kind == "near":
        X[100:140] = X[:40] + np.float32(1e-3)
        X[5000:5100] = X[4999] * np.float32(1.001)
    Xt = torch.from_numpy(X).cuda()
    D = smx.edm_packed(Xt)
    R = smx.edm_packed(Xt, ws=torch.empty(32768, dtype=torch.uint8, device="cuda"))
    if d > 8192:
        assert smx.workspace_bytes(1, n, d) == 32768 and torch.equal(D, R)
    err = [0.0, 0.0]
    for i in (0, 1, 31, 127, 128, 2500, 4995, n - 2, n - 1):
        ref = oracle.edm_rows(X, i, i + 1)
        rows = [_row(T, n, i) for T in (D, R)]
        assert rows[0][0] == rows[1][0] == 0.0
        if len(ref) > 1:
            rel = [np.abs(r[1:] - ref[1:]) / ref[1:] for r in rows]
            for q in range(2):
                err[q] += float(np.square(rel[q]).sum())
            assert ((rel[0] <= 1e-5) | (rows[0][1:] == rows[1][1:])).all()
    assert np.sqrt(err[0]) <= 1.1 * np.sqrt(err[1])
