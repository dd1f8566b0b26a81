"""All the steps of a small explicit FP64 operator in one launch (n <= 128): at
the edges of its 16-row tiles, of the lanes' elements and of its groups of 16
probes, resumed in the middle, and after breakdowns, against the oracle."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reorth", [False, True])
@pytest.mark.parametrize("dims,a,b,K,m", [
    ((2, 2, 5), (0,), (1,), 1, 3),                  # n = 4
    ((3, 5, 4), (0,), (1,), 16, 8),                 # n = 15: one row short of a tile
    ((4, 4, 3, 2), (0,), (1,), 17, 9),              # n = 16: one probe past a group
    ((3, 3, 7, 5), (0, 2), (1,), 3, 12),            # n = 63
    ((8, 8, 9), (1,), (0,), 33, 12),                # n = 64
    ((5, 13, 8), (0,), (1,), 5, 12),                # n = 65: two elements per lane, one in the second
    ((7, 17, 6), (1,), (0,), 15, 12),               # n = 119: 15 bricks
    ((2, 4, 4, 4, 6), (0, 3), (1, 2), 16, 12),      # n = 128: the product's two splits
    ((3, 43, 4), (0,), (1,), 4, 12),                # n = 129: the general kernels
])
def test_recurrence(dev, dims, a, b, K, m, reorth):
    # both sides carry rounding errors of eps times the operator's norm a step,
    # which without reorthogonalisation grow with the loss of orthogonality
    # over these few steps by less than 1e4: 1e-11 of the largest coefficient
    import torch
    from oracle import slq
    psi = ti.haar_state_dims(list(dims), 5)
    g = T.tnslq_logneg_dims(torch.from_numpy(psi).to(dev), list(dims), list(a), list(b), K, m, reorth=reorth,
                            precision="fp64", seed=2)
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), K, m, seed=2, reorth=reorth)
    big = np.abs(o["alpha"]).max()
    assert g["explicit_operator"] == 1
    assert np.abs(g["alpha"] - o["alpha"]).max() <= 1e-11 * big
    assert np.abs(g["beta"][:, 1:] - o["beta"][:, 1:]).max() <= 1e-11 * big
    assert g["n_contract_launches"] == g["n_matvecs"] == m


@pytest.mark.parametrize("reorth", [False, True])
@pytest.mark.parametrize("rule", ["diff", "fit"])
def test_resumed_steps_are_the_same(dev, rule, reorth):
    # a target that is never met: the first launch goes up to the first check,
    # the following ones take a step each
    import torch
    psi = torch.from_numpy(ti.haar_state(12, 7)).to(dev)
    args = (psi, 12, [0, 1, 2, 3], [4, 5, 6], 20, 24)
    one = T.tnslq_logneg(*args, reorth=reorth, precision="fp64", seed=3)
    many = T.tnslq_logneg(*args, reorth=reorth, precision="fp64", seed=3, stop_tol=1e-300, stop_rule=rule)
    assert many["steps_done"] == 24
    for f in ("alpha", "beta", "F", "steps"):
        assert np.array_equal(one[f], many[f])


def test_breakdown_stops_a_probe(dev):
    # A and B pure together: rho^{T_B} of a maximally entangled pair has the
    # eigenvalues +-1/d, so every probe breaks down after two steps
    import torch
    d = 8
    psi = np.zeros((d, d, 2), complex)
    psi[np.arange(d), np.arange(d), 0] = d ** -0.5
    r = T.tnslq_logneg_dims(torch.from_numpy(psi.reshape(-1)).to(dev), [d, d, 2], [0], [1], 18, 6, precision="fp64")
    assert (r["steps"] <= 2).all() and (r["alpha"][:, 2:] == 0).all() and (r["beta"][:, 3:] == 0).all()
    assert abs(r["logneg"] - 3) <= 1e-12
