"""The routes of a Lanczos step of short vectors against each other, bit for bit:
all steps in one launch (up to 64 probes, whose general product has the same order
of terms), the rest of a step in one kernel, the general kernels; and against the
oracle at the edges of the second (blocks times waves per block at most 16, which
depends on n and on the number of probes)."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,a,b,K", [
    ((3, 5, 4), (0,), (1,), 16),          # n = 15
    ((8, 8, 9), (1,), (0,), 33),          # n = 64
    ((7, 11, 6), (0,), (1,), 5),          # n = 77
    ((7, 17, 6), (1,), (0,), 64),         # n = 119
    ((2, 4, 4, 4, 6), (0, 3), (1, 2), 16),   # n = 128: two splits
])
def test_steps_in_one_launch(dev, dims, a, b, K):
    # reorthogonalised runs of more than 64 steps take a kernel or more per step
    import torch
    psi = torch.from_numpy(ti.haar_state_dims(list(dims), 5)).to(dev)
    run = {m: T.tnslq_logneg_dims(psi, list(dims), list(a), list(b), K, m, reorth=True, precision="fp64", seed=2)
           for m in (64, 65)}
    assert np.array_equal(run[64]["alpha"], run[65]["alpha"][:, :64])
    assert np.array_equal(run[64]["beta"], run[65]["beta"][:, :65])


@pytest.mark.parametrize("reorth", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("na,nb,nE,m", [(4, 4, 2, 20), (5, 5, 1, 12)])   # n = 256, 1024
def test_rest_of_a_step(dev, na, nb, nE, m, prec, reorth):
    # more than 512 probes take the general kernels; a probe's numbers do not depend
    # on how many there are
    import torch
    L = na + nb + nE
    psi = torch.from_numpy(ti.haar_state(L, 7)).to(dev)
    a, b = list(range(na)), list(range(na, na + nb))
    run = {K: T.tnslq_logneg(psi, L, a, b, K, m, reorth=reorth, precision=prec, seed=3, operator="lazy")
           for K in (512, 513)}
    for f in ("alpha", "beta", "F", "steps"):
        assert np.array_equal(run[512][f], run[513][f][:512]), f


@pytest.mark.parametrize("reorth", [False, True])
@pytest.mark.parametrize("dims,a,b,K,m", [
    ((20, 35, 3), (0,), (1,), 3, 9),       # n = 700: five blocks of three waves
    ((13, 59, 3), (1,), (0,), 2, 9),       # n = 767: the same, 153 or 154 elements each
    ((24, 32, 3), (0,), (1,), 2, 9),       # n = 768: six blocks, 12 units
    ((22, 35, 3), (0,), (1,), 2, 9),       # n = 770: six blocks of three waves, the general kernels
    ((28, 32, 3), (0,), (1,), 2, 9),       # n = 896: seven blocks, 14 units
    ((30, 30, 2), (0,), (1,), 300, 3),     # n = 900: seven blocks of three waves, the general kernels
    ((30, 30, 2), (0,), (1,), 512, 3),     # four blocks of four waves
    ((25, 40, 2), (0,), (1,), 512, 3),     # n = 1000
])
def test_edges(dev, dims, a, b, K, m, reorth):
    # the bar of the other recurrence tests: eps times the operator's norm a step,
    # grown by less than 1e4
    import torch
    from oracle import slq
    psi = ti.haar_state_dims(list(dims), 6)
    g = T.tnslq_logneg_dims(torch.from_numpy(psi).to(dev), list(dims), list(a), list(b), K, m, reorth=reorth,
                            precision="fp64", seed=4)
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), K, m, seed=4, reorth=reorth)
    big = np.abs(o["alpha"]).max()
    assert np.abs(g["alpha"] - o["alpha"]).max() <= 1e-11 * big
    assert np.abs(g["beta"][:, 1:] - o["beta"][:, 1:]).max() <= 1e-11 * big
