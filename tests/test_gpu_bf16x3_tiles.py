"""The split-BF16 contraction on the first contraction's brick output (staged
through LDS, rows of one environment index by rows) at the edges of its loop
bodies and of the output, against the oracle or, where that is too large,
complex128 products by torch.  Bar: 3e-5 norm-wise, as the parity tests (four
operands of 16 significant bits)."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu


# d_A from one brick (32 terms) to 16: 3 to 48 phases, bodies of 6; columns on
# and off half a tile; d_B below 8 (direct stores) and above
@pytest.mark.parametrize("na,nb,nE,K", [(5, 3, 3, 9), (5, 5, 2, 3), (6, 4, 3, 5), (7, 2, 4, 21), (7, 6, 1, 2),
                                        (8, 5, 2, 7), (8, 3, 0, 40), (3, 3, 6, 13)])
def test_short_runs(dev, na, nb, nE, K):
    import torch
    L = na + nb + nE
    a, b = list(range(nE, nE + na)), list(range(nE + na, L))
    psi = ti.haar_state(L, 21)
    X = ti.random_vectors(K, 1 << (na + nb), seed=22)
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision="bf16x3")
    ref = exact.pt_matvec_lazy(exact.regroup(psi, L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= 3e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("na,nb,nE,K", [(9, 5, 6, 512), (10, 5, 5, 512)])
def test_longer_runs(dev, na, nb, nE, K):
    # 16 and 32 bricks with enough tiles that the first contraction is not split
    import torch
    L = na + nb + nE
    a, b = list(range(nE, nE + na)), list(range(nE + na, L))
    psi = ti.haar_state_torch(L, 23, dev, torch.complex128)
    X = ti.random_vectors_torch(K, 1 << (na + nb), 24, dev)
    Y = T.tnslq_ptmatvec(psi, L, a, b, X, precision="bf16x3")
    P = psi.reshape(1 << nE, 1 << na, 1 << nb)
    ref = torch.zeros_like(X).reshape(K, 1 << na, 1 << nb)
    for k in range(0, K, 64):
        x = X[k:k + 64].reshape(64, 1 << na, 1 << nb)
        for M in P:
            # Ups[k][b'][b] = sum_a' X[k][a'][b'] conj M[a'][b];  Y[k][a][b] += sum_b' M[a][b'] Ups[k][b'][b]
            u = (x.transpose(1, 2).reshape(64 << nb, 1 << na).contiguous() @ M.conj().contiguous()).reshape(64, 1 << nb, 1 << nb)
            y = M @ u.transpose(0, 1).reshape(1 << nb, 64 << nb).contiguous()
            ref[k:k + 64] += y.reshape(1 << na, 64, 1 << nb).transpose(0, 1)
    err = torch.linalg.vector_norm(Y - ref.reshape(K, -1)) / torch.linalg.vector_norm(ref)
    assert float(err) <= 3e-5
