"""The split-BF16 contraction where a block walks several tiles (more than 256 of
them, runs of at most 32 bricks) and a run is no multiple of the loop body (12
phases, 4 bricks): the buffers start anew for every tile, 1, 2 or 3 bricks into a
body.  Against complex128 products.  Bar: 3e-5 norm-wise, as the parity tests."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti

pytestmark = pytest.mark.gpu


# d_A = 32 or 64: one or two bricks in the first contraction, 512 tiles of it or
# more, the last column of tiles whole or half empty
@pytest.mark.parametrize("na,nb,nE,K", [(5, 5, 5, 256), (6, 5, 5, 256), (5, 4, 7, 300), (6, 6, 3, 300)])
def test_first_contraction(dev, na, nb, nE, K):
    import torch
    L = na + nb + nE
    assert -(-(1 << (nb + nE)) // 128) * -(-(K << nb) // 128) > 256
    a, b = list(range(nE, nE + na)), list(range(nE + na, L))
    psi = ti.haar_state_torch(L, 23, dev, torch.complex128)
    X = ti.random_vectors_torch(K, 1 << (na + nb), 24, dev)
    Y = T.tnslq_ptmatvec(psi, L, a, b, X, precision="bf16x3")
    P = psi.reshape(1 << nE, 1 << na, 1 << nb)
    ref = torch.zeros_like(X).reshape(K, 1 << na, 1 << nb)
    x = X.reshape(K, 1 << na, 1 << nb)
    for M in P:
        # Ups[k][b'][b] = sum_a' X[k][a'][b'] conj M[a'][b];  Y[k][a][b] += sum_b' M[a][b'] Ups[k][b'][b]
        u = (x.transpose(1, 2).reshape(K << nb, 1 << na).contiguous() @ M.conj().contiguous()).reshape(K, 1 << nb, 1 << nb)
        y = M @ u.transpose(0, 1).reshape(1 << nb, K << nb).contiguous()
        ref += y.reshape(1 << na, K, 1 << nb).transpose(0, 1)
    ref = ref.reshape(K, -1)
    # every vector: a stale buffer spoils one tile's
    err = torch.linalg.vector_norm(Y - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)
    assert float(err.max()) <= 3e-5


# the operator formed over d_E = 65 .. 96 environment terms (3 bricks), and 129 .. 160
# (5), in 18 x 18 tiles: the first two coefficients of every probe against FP64's,
# each a bilinear form of the operator with a 3e-5 bar
@pytest.mark.parametrize("dE", [70, 96, 150])
def test_formed_operator(dev, dE):
    import torch
    dims = [48, 48, dE]
    psi = torch.from_numpy(ti.haar_state_dims(dims, 9)).to(dev)
    run = {p: T.tnslq_logneg_dims(psi, dims, [0], [1], 128, 1, precision=p, seed=3) for p in ("fp64", "bf16x3")}
    assert run["bf16x3"]["explicit_operator"] == 1
    x, y = run["bf16x3"], run["fp64"]
    big = np.hypot(y["alpha"][:, 0], y["beta"][:, 1])
    assert (np.abs(x["alpha"][:, 0] - y["alpha"][:, 0]) <= 6e-5 * big).all()
    assert (np.abs(x["beta"][:, 1] - y["beta"][:, 1]) <= 6e-5 * big).all()
