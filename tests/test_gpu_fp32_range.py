"""The FP32 block matvec over the whole range of FP32: vectors and states far
below one (where BF16 pieces of a value no longer add up to it), at the top of the
range (where Re + Im, or a value rounded to BF16, is infinite), vectors of
different sizes in one call, zero and non-finite ones; in tiles of few columns
and in large ones, a vector being part of a column tile or several.  Against the
oracle; 1e-6 of each vector's result, the bar of ordinary values."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu

# K d_B = 36, 40, 64, 64 columns, then 80, 96, 160, 256; d_B from 4 to 128
SHAPES = [(14, 9, 2, 9), (12, 7, 3, 5), (15, 10, 5, 2), (14, 6, 6, 1), (13, 6, 4, 5), (16, 9, 5, 3), (12, 5, 2, 40),
          (15, 7, 7, 2)]


def matvec(dev, L, na, nb, psi, X):
    import torch
    a, b = list(range(L - na - nb, L - nb)), list(range(L - nb, L))
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision="fp32")
    return Y.cpu().numpy(), lambda psi, X: exact.pt_matvec_lazy(exact.regroup(psi, L, a, b), X)


def inputs(L, na, nb, K):
    """A state and vectors of largest entry one."""
    psi = ti.haar_state(L, 3)
    X = ti.random_vectors(K, 1 << (na + nb), seed=4)
    return psi / np.abs(psi).max(), X / np.abs(X).max()


def errors(Y, ref, scale=1.0):
    """Per vector, of the result (scaled by a power of two, so that its square is in range)."""
    s = 2.0 ** -np.floor(np.log2(scale))
    return np.linalg.norm((Y - ref) * s, axis=1) / np.linalg.norm(ref * s, axis=1)


# 1e-38: FP32's subnormals, whose unit (1.4e-45) is 6e-7 of these vectors'
# entries; some 200 roundings to it in the two sums, at random: below 5e-6
@pytest.mark.parametrize("xs,ps,tol", [(1e-34, 1.0, 1e-6), (1e-36, 1.0, 1e-6), (1e-38, 1.0, 5e-6), (1e36, 1e-35, 1e-6)])
@pytest.mark.parametrize("L,na,nb,K", SHAPES)
def test_small_values(dev, L, na, nb, K, xs, ps, tol):
    psi, X = inputs(L, na, nb, K)
    Y, ref = matvec(dev, L, na, nb, psi * ps, X * xs)
    assert (errors(Y, ref(psi, X) * (xs * ps ** 2), xs * ps ** 2) <= tol).all()


@pytest.mark.parametrize("L,na,nb,K", SHAPES)
def test_vectors_of_different_sizes(dev, L, na, nb, K):
    psi, X = inputs(L, na, nb, K)
    size = np.array([(1e-36, 1.0, 1e-33, 1e20, 0.0)[k % 5] for k in range(K)])[:, None]
    Y, ref = matvec(dev, L, na, nb, psi, X * size)
    some = size[:, 0] > 0
    size = size[some]
    assert (errors(Y[some] / size, ref(psi, X)[some]) <= 1e-6).all()
    assert (Y[~some] == 0).all()


# 3.4e38 is below FP32's largest value and above the largest that rounds to a
# finite BF16; 2e38 is finite there, but not twice it.  A unit state of 2^L
# entries makes of either results below 1e38.
@pytest.mark.parametrize("xs", [2e38, 3.4e38])
@pytest.mark.parametrize("L,na,nb,K", SHAPES)
def test_largest_values(dev, L, na, nb, K, xs):
    psi = ti.haar_state(L, 3)
    X = ti.random_vectors(K, 1 << (na + nb), seed=4)
    X = np.sign(X.real) + 1j * np.sign(X.imag)
    Y, ref = matvec(dev, L, na, nb, psi, X * xs)
    r = ref(psi, X)
    assert np.abs(r).max() * xs < 1e38
    assert (errors(Y / xs, r) <= 1e-6).all()


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("L,na,nb,K", [s for s in SHAPES if s[3] > 1])
def test_non_finite_vector_stays_apart(dev, L, na, nb, K, bad):
    psi, X = inputs(L, na, nb, K)
    ref = matvec(dev, L, na, nb, psi, X)[1](psi, X)
    X[1, 5] = bad
    Y = matvec(dev, L, na, nb, psi, X)[0]
    assert not np.isfinite(Y[1]).any()
    rest = np.arange(K) != 1
    assert (errors(Y[rest], ref[rest]) <= 1e-6).all()
