"""The sum of a block matvec's split partials, in the caller's order with the
roles of A and B kept and exchanged, for few and many splits, against the
oracle.  Bars: the parity tests'."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-6)])
@pytest.mark.parametrize("L,a,b,K", [
    (8, [0, 1], [2, 3, 4, 5], 3),                          # n = 64: less than a block; one split
    (13, [1, 2, 3], [4, 5, 6, 7, 8, 9], 5),                # exchanged, n = 512
    (13, [4, 5, 6, 7, 8, 9], [1, 2, 3], 5),                # as given
    (18, [0, 1, 2, 3], [6, 7, 8, 9, 10], 9),               # exchanged, a long environment: many splits
    (18, [6, 7, 8, 9, 10], [0, 1, 2, 3], 9),
])
def test_matvec(dev, prec, tol, L, a, b, K):
    import torch
    psi = ti.haar_state(L, 8)
    X = ti.random_vectors(K, 1 << (len(a) + len(b)), seed=9)
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision=prec)
    ref = exact.pt_matvec_lazy(exact.regroup(psi, L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
