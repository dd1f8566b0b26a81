"""The FP32 product of few columns in BF16 pieces: steps of two 16-term bricks at
odd and even counts, restarts every four steps, column tiles of 16, and values
that need all three pieces; through the explicit operator's first steps and the
lazy matvec, against the oracle."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,a,b,K", [
    ((3, 5, 7), (0,), (1,), 1),              # n = 15: one brick, not full
    ((4, 4, 9), (0,), (1,), 16),             # n = 16: one brick, half a step
    ((6, 8, 5), (0,), (1,), 17),             # n = 48: a step and a half
    ((9, 16, 3), (1,), (0,), 33),            # n = 144: 9 bricks, past a restart
    ((11, 31, 3), (0,), (1,), 48),           # n = 341: 22 bricks, the last not full
    ((21, 64, 2), (0,), (1,), 64),           # n = 1344: 84 bricks in splits
])
def test_explicit(dev, dims, a, b, K):
    # alpha_1 and beta_2 of every probe: one product of the operator (1e-6 of its
    # result at most, as the matvec's bar) on an operator formed to as much
    import torch
    from oracle import slq
    psi = ti.haar_state_dims(list(dims), 3)
    g = T.tnslq_logneg_dims(torch.from_numpy(psi).to(dev), list(dims), list(a), list(b), K, 1, precision="fp32", seed=8)
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), K, 1, seed=8)
    big = np.hypot(o["alpha"][:, 0], o["beta"][:, 1])
    assert (np.abs(g["alpha"][:, 0] - o["alpha"][:, 0]) <= 2e-6 * big).all()
    assert (np.abs(g["beta"][:, 1] - o["beta"][:, 1]) <= 2e-6 * big).all()


@pytest.mark.parametrize("scale", [1.0, 1e-12, 1e12])
@pytest.mark.parametrize("L,a,b,K", [
    (12, [1, 2, 3, 4, 5, 6, 7], [8], 5),               # 8 bricks, 10 columns
    (14, [0, 1, 2, 3, 4, 5, 6, 7, 8], [10, 11], 9),    # 36 columns
    (15, [2, 3, 4, 5, 6, 7, 8, 9, 10, 11], [0, 1, 12], 7),   # 56 columns
])
def test_lazy_matvec(dev, L, a, b, K, scale):
    # scaled vectors: the pieces' exponents move with the value
    import torch
    psi = ti.haar_state(L, 3)
    X = ti.random_vectors(K, 1 << (len(a) + len(b)), seed=4) * scale
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision="fp32")
    ref = exact.pt_matvec_lazy(exact.regroup(psi, L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= 1e-6 * np.linalg.norm(ref)
