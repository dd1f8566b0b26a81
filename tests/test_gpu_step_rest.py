"""The rest of a step of short vectors in one kernel: at the edges of its units
(blocks of 128 to 255 elements in waves of 64, 16 waves at most), on both sides
of the bound on reorthogonalised steps, in FP64 and FP32, explicit and lazy,
against the oracle."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reorth", [False, True])
@pytest.mark.parametrize("dims,a,b,K,m", [
    ((3, 43, 4), (0,), (1,), 2, 9),                # n = 129: one block of three units
    ((5, 51, 6), (1,), (0,), 9, 12),               # n = 255: one block of 255
    ((16, 16, 6), (0,), (1,), 3, 12),              # n = 256: two blocks of two whole units
    ((13, 29, 5), (0,), (1,), 4, 9),               # n = 377
    ((9, 71, 4), (0,), (1,), 3, 28),               # n = 639: 4 blocks of 160; steps past the bound
    ((20, 32, 3), (0,), (1,), 2, 9),               # n = 640: 5 blocks, 10 units
    ((31, 33, 2), (0,), (1,), 2, 6),               # n = 1023: 21 units, the general kernels
    ((32, 32, 3), (0,), (1,), 2, 19),              # n = 1024: 16 units; steps past the bound
])
def test_recurrence_fp64(dev, dims, a, b, K, m, reorth):
    # the bar of the small operators' test: rounding errors of eps times the
    # operator's norm a step, without reorthogonalisation grown by the loss of
    # orthogonality over at most 28 steps on these spectra by less than 1e4
    import torch
    from oracle import slq
    m = m if reorth else min(m, 12)
    psi = ti.haar_state_dims(list(dims), 6)
    g = T.tnslq_logneg_dims(torch.from_numpy(psi).to(dev), list(dims), list(a), list(b), K, m, reorth=reorth,
                            precision="fp64", seed=4)
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), K, m, seed=4, reorth=reorth)
    big = np.abs(o["alpha"]).max()
    assert np.abs(g["alpha"] - o["alpha"]).max() <= 1e-11 * big
    assert np.abs(g["beta"][:, 1:] - o["beta"][:, 1:]).max() <= 1e-11 * big


@pytest.mark.parametrize("operator", ["explicit", "lazy"])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 2e-5), ("bf16x3", 6e-4)])
def test_forms_and_precisions(dev, operator, prec, tol):
    # one step's product is off by 1e-6 (FP32) or 3e-5 (split BF16) of the
    # result at most, as in the matvec tests; 20 times that over 6 steps
    import torch
    from oracle import slq
    L, a, b = 13, [1, 2, 3, 4], [6, 7, 8, 9, 10]
    psi = ti.haar_state(L, 6)
    g = T.tnslq_logneg(torch.from_numpy(psi).to(dev), L, a, b, 5, 6, reorth=True, precision=prec, seed=4,
                       operator=operator)
    o = slq.slq_logneg(psi, L, a, b, 5, 6, seed=4, reorth=True)
    big = np.abs(o["alpha"]).max()
    assert np.abs(g["alpha"] - o["alpha"]).max() <= tol * big
    assert np.abs(g["beta"][:, 1:] - o["beta"][:, 1:]).max() <= tol * big


def test_breakdown_stops_a_probe(dev):
    import torch
    d = 16
    psi = np.zeros((d, d, 2), complex)
    psi[np.arange(d), np.arange(d), 0] = d ** -0.5
    for reorth in (False, True):
        r = T.tnslq_logneg_dims(torch.from_numpy(psi.reshape(-1)).to(dev), [d, d, 2], [0], [1], 3, 6, reorth=reorth,
                                precision="fp64")
        assert (r["steps"] <= 2).all() and (r["alpha"][:, 2:] == 0).all() and (r["beta"][:, 3:] == 0).all()
        assert abs(r["logneg"] - 4) <= 1e-12
