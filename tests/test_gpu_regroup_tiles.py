"""psi regrouped into the streaming forms' copies in one read (tiles of 2^12 or
2^13 amplitudes): sizes on both sides of a tile, qubit orders that put psi's and
the copies' lowest bits together, apart and interleaved, states off a 16-byte
boundary; and the norm that is taken from the same read.  Oracle: the lazy
matvec in complex128; FP64 products and sums, the parity tests' bar of 1e-12."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu


def _tensor(psi, dtype, dev, offset):
    import torch
    t = torch.zeros(psi.size + offset, dtype=getattr(torch, dtype), device=dev)
    t[offset:] = torch.from_numpy(psi).to(dev)
    return t[offset:]


@pytest.mark.parametrize("dtype", ["complex64", "complex128"])
@pytest.mark.parametrize("L,a,b,K,offset", [
    (11, [0, 1, 2, 3], [4], 1, 0),                           # below a tile
    (12, [11, 2, 5], [0], 3, 0),                             # one tile in complex128
    (13, [0, 1, 2, 3, 4, 5], [6, 7], 2, 1),                  # one tile in complex64; off 16 bytes
    (14, [8, 9, 10, 11, 12, 13], [0, 1, 2], 1, 0),           # psi's lowest bits in A
    (15, [14, 0, 13, 1, 12, 2, 11, 3], [7], 4, 1),           # interleaved from both ends
    (17, [1, 3, 5, 7, 9, 11, 13, 15], [0, 16, 8], 1, 0),     # every other qubit, B at both ends
    (18, [4, 5, 6, 7, 8, 9, 10, 11, 12, 13], [], 5, 0),      # rows of one operand wide of a panel
    (20, [2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12], [13], 1, 0),  # one read of psi in complex64
])
def test_matvec(dev, dtype, L, a, b, K, offset):
    import torch
    psi = ti.haar_state(L, 5).astype(dtype)
    if not b:
        b = [L - 1]
    X = ti.random_vectors(K, 1 << (len(a) + len(b)), seed=6)
    Y = T.tnslq_ptmatvec(_tensor(psi, dtype, dev, offset), L, a, b, torch.from_numpy(X).to(dev), precision="fp64")
    ref = exact.pt_matvec_lazy(exact.regroup(psi.astype(np.complex128), L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("dtype,off", [("complex64", 3e-3), ("complex128", 1e-4)])
@pytest.mark.parametrize("L", [11, 13, 22])
@pytest.mark.parametrize("at", [0, 1, 5000, -1])
def test_state_check(dev, dtype, off, L, at):
    # 22 qubits: 512 or 1024 tiles, two or one for each block; off the norm by
    # more than its tolerance (1e-4 in complex64, 1e-9 in complex128)
    psi = np.zeros(1 << L, dtype)
    at = at % (1 << L)
    psi[at] = 1.0
    other = (at + 77) % (1 << L)
    runs = (lambda t: T.tnslq_spectral_sum(t, L, [0, 1, 2], "purity", 1, 2),
            lambda t: T.tnslq_logneg(t, L, [1, 2, 3, 4, 5, 6, 7], [0], 1, 2, precision="fp64", operator="lazy"))
    for run in runs:
        run(_tensor(psi, dtype, dev, 0))
        for value, status in ((np.nan, T.TNSLQ_E_NONFINITE), (np.inf, T.TNSLQ_E_NONFINITE),
                              (off ** 0.5, T.TNSLQ_E_STATE)):
            bad = psi.copy()
            bad[other] = value
            with pytest.raises(T.TnslqError) as e:
                run(_tensor(bad, dtype, dev, 0))
            assert e.value.status == status
