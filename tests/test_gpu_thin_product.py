"""Products with few columns (16-row tiles against all columns) at the edges
of their tiles and splits, against the oracle."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact, slq

pytestmark = pytest.mark.gpu


# K d_B from 9 (past the streaming form) to 64 columns, and just past them
@pytest.mark.parametrize("prec,tol", [("fp32", 1e-6), ("fp64", 1e-12)])
@pytest.mark.parametrize("L,a,b,K", [
    (8, [0, 1, 2], [4, 5], 3),                 # 12 columns, d_A below one tile of rows
    (10, [3, 4, 5, 6], [0], 8),                # 16: one column tile exactly
    (11, [0, 2, 4, 6], [1], 9),                # 18: two column tiles, the second nearly empty
    (12, [5, 6, 7, 8, 9], [1, 2], 11),         # 44
    (13, [0, 1, 2, 3, 4, 5], [8, 9, 10], 8),   # 64: the last thin shape
    (13, [0, 1, 2, 3, 4, 5], [8, 9, 10], 9),   # 72: the first of 128-column tiles
    (13, [0, 1, 2, 3], [9, 10, 11], 24),       # 192 columns over 16 terms (FP64: groups of 64 columns)
    (9, [0, 1], [2, 3, 4, 5], 5),              # roles exchanged, 20 columns
])
def test_matvec_with_few_columns(dev, prec, tol, L, a, b, K):
    import torch
    psi = ti.haar_state(L, 3)
    X = ti.random_vectors(K, 1 << (len(a) + len(b)), seed=4)
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision=prec)
    ref = exact.pt_matvec_explicit(exact.regroup(psi, L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)


# the explicit operator: n off every tile and brick size, runs of bricks of
# unequal length, one column to past the limit.  Bars of the explicit form:
# 1e-10 of the largest coefficient in FP64, 1e-4 of the estimate in FP32.
@pytest.mark.parametrize("K", [1, 16, 17, 64, 65])
@pytest.mark.parametrize("dims,a,b", [((3, 5, 7, 4), (0,), (1,)), ((5, 7, 3, 9, 4), (0, 3), (1, 2))])
def test_explicit_operator_with_few_probes(dev, dims, a, b, K):
    import torch
    psi = ti.haar_state_dims(list(dims), 8)
    t = torch.from_numpy(psi).to(dev)
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), min(K, 5), 7, seed=1, reorth=True)
    g = T.tnslq_logneg_dims(t, list(dims), list(a), list(b), K, 7, reorth=True, precision="fp64", seed=1)
    big = np.abs(o["alpha"]).max()
    k = min(K, 5)
    assert np.abs(g["alpha"][:k] - o["alpha"]).max() <= 1e-10 * big
    assert np.abs(g["beta"][:k, 1:] - o["beta"][:, 1:]).max() <= 1e-10 * big
    f = T.tnslq_logneg_dims(t, list(dims), list(a), list(b), K, 7, reorth=True, precision="fp32", seed=1)
    assert abs(f["logneg"] - g["logneg"]) <= 1e-4 * max(abs(g["logneg"]), 1.0)
