"""The Lanczos kernels at the edges of their wave and block layouts, through
the entry points, against the oracle."""
import numpy as np
import pytest

import paper_1809_01685_amd as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e-200, 1e150])
@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 128])
def test_quadrature_at_wave_edges(dev, m, scale):
    # one wave holds up to 64 entries in one register per lane, up to 128 in
    # two; rows: random, with zero couplings (split matrices), all zero, cut
    # short by `steps`.  Tolerance: implicit QL leaves each entry a backward
    # error of at most about 8 m eps |T| (1.7 m rotations of a few roundings
    # each), x -> |x| changes by at most about 3 times the perturbation
    # ((2 / pi) log m + 1), and both sides carry it.
    import torch
    rng = np.random.default_rng(m)
    K = 6
    al = rng.standard_normal((K, m)) * scale
    be = np.abs(rng.standard_normal((K, m + 1))) * scale
    be[2, 1:m:3] = 0.0
    al[3], be[3] = 0.0, 0.0
    al[4] = scale                      # equal diagonal entries, weak couplings
    be[4, 1:] *= 1e-9
    steps = np.full(K, m, dtype=np.int32)
    steps[5] = (m + 1) // 2
    F = T.tnslq_quadrature(torch.from_numpy(al).to(dev), torch.from_numpy(be).to(dev),
                           torch.from_numpy(steps).to(dev)).cpu().numpy()
    for k in range(K):
        for j in range(1, m + 1):
            jj = min(j, steps[k])
            t = np.diag(al[k, :jj]) + np.diag(be[k, 1:jj], 1) + np.diag(be[k, 1:jj], -1)
            lam, v = np.linalg.eigh(t / scale)
            want = float((v[0] ** 2 * np.abs(lam)).sum())
            norm = max(np.abs(lam).max(), 1e-300)
            assert abs(F[k, j - 1] / scale - want) <= 48 * m * np.finfo(float).eps * norm, (k, j)


@pytest.mark.parametrize("dims,a,b,K,m", [
    ((2, 2, 3, 4), (0,), (1,), 3, 2),                  # n = 4: one chunk, mostly empty lanes
    ((3, 3, 7, 6), (0, 2), (1,), 5, 9),                # n = 63: one element short of a wave
    ((5, 13, 4, 5), (0,), (1,), 600, 12),              # n = 65, 600 probes: 128-element chunks
    ((2, 2, 2, 5, 9, 3, 8), (0, 3, 4), (1, 2, 5), 4, 40),   # n = 1080: 17 chunks, added by their readers
    ((2, 3, 7, 3, 19, 3), (1, 2, 4), (0, 3), 2, 33),   # n = 2394: 38 chunks, added by a kernel
])
def test_reorthogonalised_recurrence_at_chunk_edges(dev, dims, a, b, K, m):
    # alpha, beta and the basis they come from: against a recurrence in 64
    # bits that orthogonalises twice, from the explicit operator.  Both sides
    # are backward stable with an orthonormal basis, so the coefficients agree
    # to a modest multiple of eps times the operator's norm: 1e-11 of the
    # largest, as the parity tests of the explicit form.
    import torch
    import tnslq_inputs as ti
    from oracle import slq
    psi = ti.haar_state_dims(list(dims), 5)
    g = T.tnslq_logneg_dims(torch.from_numpy(psi).to(dev), list(dims), list(a), list(b), K, m, reorth=True,
                            precision="fp64", seed=2)
    Ko = min(K, 6)   # the oracle's first probes are the same ones
    o = slq.slq_logneg_dims(psi, list(dims), list(a), list(b), Ko, m, seed=2, reorth=True)
    big = np.abs(o["alpha"]).max()
    assert np.abs(g["alpha"][:Ko] - o["alpha"]).max() <= 1e-11 * big
    assert np.abs(g["beta"][:Ko, 1:] - o["beta"][:, 1:]).max() <= 1e-11 * big
