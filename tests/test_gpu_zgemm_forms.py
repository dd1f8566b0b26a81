"""The MPS matvec's complex products on both sides of their switch to three
real products (64 terms), in whole and cut tiles: estimates on small chains
against the oracle's explicit operator, coefficient by coefficient."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import mps, slq

pytestmark = pytest.mark.gpu


# (sites, bond, A, B): reductions k_A, k_B, U'M and M V around 64, tiles of 64
# outputs cut (bonds 7, 9) and whole (8, 16); factors (adjacent) and network (gap)
@pytest.mark.parametrize("L,chi,a0,la,b0,lb", [(12, 7, 4, 4, 8, 3), (14, 8, 4, 6, 10, 3), (14, 9, 4, 4, 9, 4),
                                               (14, 16, 4, 6, 10, 3), (16, 8, 5, 3, 9, 4)])
@pytest.mark.parametrize("matvec", ["factors", "network"])
def test_products_match_oracle(dev, L, chi, a0, la, b0, lb, matvec):
    ts = ti.random_mps(L, 2, chi, 3)
    K, m = 5, 6
    g = T.tnslq_logneg_mps(ts, a0, la, b0, lb, K, m, device=dev, reorth=True, seed=4, matvec=matvec)
    psi = mps.mps_to_dense(ts)
    psi = psi / np.linalg.norm(psi)
    if 2 ** la > ts[a0].shape[0] * ts[a0 + la].shape[0] or 2 ** lb > ts[b0].shape[0] * (
            ts[b0 + lb].shape[0] if b0 + lb < L else 1):
        pytest.skip("compressed blocks: the probes live in another basis")
    o = slq.slq_logneg(psi, L, list(range(a0, a0 + la)), list(range(b0, b0 + lb)), K, m, seed=4, reorth=True)
    big = np.abs(o["alpha"]).max()
    # the bar of the factorised operator's parity tests
    assert np.abs(g["alpha"] - o["alpha"]).max() <= 1e-10 * big
    assert np.abs(g["beta"][:, 1:] - o["beta"][:, 1:]).max() <= 1e-10 * big
