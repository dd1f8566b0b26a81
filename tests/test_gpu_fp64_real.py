"""Rounding of the FP64 contractions in three real products, for real and complex
states and vectors: no larger than that of four products summed one term after
the other, exact zeros where the operands are real, and no overflow where four
products have none."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu

# more than 64 columns and runs of more than 32 terms: the tiles of three products
SHAPES = [(13, 6, 4, 5), (14, 8, 4, 9), (16, 6, 6, 3), (14, 9, 3, 17)]


def inputs(L, na, nb, K, kind):
    psi = ti.haar_state(L, 3)
    X = ti.random_vectors(K, 1 << (na + nb), seed=4)
    psi = psi if kind[0] == "c" else psi.real + 0j
    return psi / np.linalg.norm(psi), X if kind[1] == "c" else X.real + 0j


def matvec(dev, L, na, nb, psi, X):
    import torch
    a, b = list(range(L - na - nb, L - nb)), list(range(L - nb, L))
    return T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev),
                            precision="fp64").cpu().numpy()


def products(A, B, real, run):
    """A B^T over complex entries: in runs of `run` terms added up one after the other, in four
    real products each, in the type `real`."""
    ar, ai, br, bi = (np.ascontiguousarray(x.T, dtype=real) for x in (A.real, A.imag, B.real, B.imag))
    re = np.zeros((A.shape[0], B.shape[0]), real)
    im = re.copy()
    for l0 in range(0, A.shape[1], run):
        r, i = np.zeros_like(re), np.zeros_like(im)
        for l in range(l0, min(l0 + run, A.shape[1])):
            r += np.outer(ar[l], br[l])
            r -= np.outer(ai[l], bi[l])
            i += np.outer(ar[l], bi[l])
            i += np.outer(ai[l], br[l])
        re += r
        im += i
    return re, im


class Parts:
    """Real and imaginary parts of any type, with the attributes that products() takes."""

    def __init__(self, re, im):
        self.real, self.imag, self.shape = re, im, re.shape


def four_products(L, na, nb, psi, X, real, run):
    """The two contractions of the block matvec."""
    dA, dB, K = 1 << na, 1 << nb, X.shape[0]
    P = psi.reshape(-1, dA, dB)
    dE = P.shape[0]
    re, im = products(P.conj().transpose(0, 2, 1).reshape(dE * dB, dA),
                      X.reshape(K, dA, dB).transpose(0, 2, 1).reshape(K * dB, dA), real, run)
    ups = [x.reshape(dE, dB, K, dB).transpose(2, 1, 0, 3).reshape(K * dB, dE * dB) for x in (re, im)]
    re, im = products(P.transpose(1, 0, 2).reshape(dA, dE * dB), Parts(*ups), real, run)
    return [x.reshape(dA, K, dB).transpose(1, 0, 2).reshape(K, -1) for x in (re, im)]


def norm(re, im):
    return float(np.sqrt((re * re).sum() + (im * im).sum()))


@pytest.mark.parametrize("kind", ["rr", "rc", "cr", "cc"])
@pytest.mark.parametrize("L,na,nb,K", SHAPES[:3])
def test_rounds_no_more_than_four_products(dev, L, na, nb, K, kind):
    # the bar: runs of 64 terms (the shortest that a contraction is split into)
    # in double, one product after the other; the reference in 80 bits
    psi, X = inputs(L, na, nb, K, kind)
    Y = matvec(dev, L, na, nb, psi, X)
    re, im = four_products(L, na, nb, psi, X, np.longdouble, 1 << 30)
    r4, i4 = four_products(L, na, nb, psi, X, np.float64, 64)
    assert norm(Y.real - re, Y.imag - im) <= norm(r4 - re, i4 - im)


@pytest.mark.parametrize("L,na,nb,K", SHAPES)
def test_real_operands_stay_real(dev, L, na, nb, K):
    psi, X = inputs(L, na, nb, K, "rr")
    Y = matvec(dev, L, na, nb, psi, X)
    assert (Y.imag == 0).all()
    ref = exact.pt_matvec_lazy(exact.regroup(psi, L, list(range(L - na - nb, L - nb)), list(range(L - nb, L))), X)
    assert np.linalg.norm(Y - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("dE", [33, 41, 56, 64, 100])   # 5 to 13 bricks: every remainder of a loop body
def test_operator_of_a_real_state_is_real(dev, dE):
    import torch
    dims = [5, 4, 3, 2, dE]
    psi = ti.haar_state_dims(dims, 4).real + 0j
    rho = T.tnslq_rho_pt_dims(torch.from_numpy(psi / np.linalg.norm(psi)).to(dev), dims, [0, 2], [1, 3]).cpu().numpy()
    P = exact.regroup_dims(psi / np.linalg.norm(psi), dims, [0, 2], [1, 3])
    want = np.einsum("abe,cde->abcd", P, P.conj()).transpose(0, 3, 2, 1).reshape(rho.shape)
    assert (rho.imag == 0).all()
    assert np.abs(rho - want).max() <= 1e-13 * np.abs(want).max()


@pytest.mark.parametrize("L,na,nb,K", SHAPES)
def test_largest_values(dev, L, na, nb, K):
    # Re + Im = 2e308 is infinite; of a unit state the results are below 1e308
    psi, X = inputs(L, na, nb, K, "cc")
    X = np.sign(X.real) + 1j * np.sign(X.imag)
    Y = matvec(dev, L, na, nb, psi, X * 1e308)
    ref = exact.pt_matvec_lazy(exact.regroup(psi, L, list(range(L - na - nb, L - nb)), list(range(L - nb, L))), X)
    assert np.abs(ref).max() < 1
    assert np.linalg.norm(Y / 1e308 - ref) <= 1e-12 * np.linalg.norm(ref)
