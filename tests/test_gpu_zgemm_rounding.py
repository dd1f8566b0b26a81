"""The MPS matvec's complex products in three real products, for real and complex
matrices: rounding no larger than that of four products summed one term after the
other, and imaginary parts of exactly zero where both are real.  The launcher is
called as the matvec calls it."""
import ctypes

import numpy as np
import pytest

import paper_1809_01685_amd as T

pytestmark = pytest.mark.gpu

# launch_zgemm(opa, opb, A, B, C, M, N, K, lda, ldb, ldc, batch, sa, sb, sc, stream, sub, ks, csk, form)
SYMBOL = "_ZN5tnslq12launch_zgemmEiiPK15HIP_vector_typeI%sLj2EES3_PS1_iiilllilllP12ihipStream_tiili"


def zgemm(dev, opa, opb, A, B, real):
    """op(A) op(B) of numpy matrices, op 0 as stored, 2 the conjugate transpose."""
    import torch
    f = getattr(T.lib(), SYMBOL % ("d" if real is np.float64 else "f"))
    i, l, p = ctypes.c_int, ctypes.c_int64, ctypes.c_void_p
    f.argtypes = [i, i, p, p, p, i, i, i, l, l, l, i, l, l, l, p, i, i, l, i]
    f.restype = i
    dtype = np.complex128 if real is np.float64 else np.complex64
    M, K = A.shape if opa == 0 else A.shape[::-1]
    N = B.shape[1] if opb == 0 else B.shape[0]
    a, b = (torch.from_numpy(np.ascontiguousarray(x, dtype=dtype)).to(dev) for x in (A, B))
    c = torch.zeros(M, N, dtype=a.dtype, device=dev)
    assert a.shape[1] >= 1 and c.is_contiguous()
    rc = f(opa, opb, a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, a.shape[1], b.shape[1], N, 1, 0, 0, 0,
           torch.cuda.current_stream().cuda_stream, 0, 1, 0, 3)
    assert rc == 0
    torch.cuda.synchronize()
    return c.cpu().numpy()


def product(a, b, real):
    """a b in four real products, the terms added up one after the other in the type `real`."""
    re = np.zeros((a.shape[0], b.shape[1]), real)
    im = re.copy()
    ar, ai, br, bi = (x.astype(real) for x in (a.real, a.imag, b.real, b.imag))
    for l in range(a.shape[1]):
        re += np.outer(ar[:, l], br[l])
        re -= np.outer(ai[:, l], bi[l])
        im += np.outer(ar[:, l], bi[l])
        im += np.outer(ai[:, l], br[l])
    return re, im


def norm(re, im):
    return float(np.sqrt((re * re).sum() + (im * im).sum()))


# 64 terms: the shortest sum that takes three products; whole and cut tiles
@pytest.mark.parametrize("real", [np.float64, np.float32])
@pytest.mark.parametrize("kind", ["rr", "rc", "cr", "cc"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (2, 0), (0, 2)])
@pytest.mark.parametrize("M,N,K", [(128, 192, 64), (150, 130, 70), (128, 128, 512)])
def test_rounds_no_more_than_four_products(dev, M, N, K, opa, opb, kind, real):
    rng = np.random.default_rng(K)

    def matrix(r, c, complex_):
        x = rng.standard_normal((r, c)) + (1j * rng.standard_normal((r, c)) if complex_ else 0)
        return x.astype(np.complex128 if real is np.float64 else np.complex64)

    a, b = matrix(M, K, kind[0] == "c"), matrix(K, N, kind[1] == "c")
    C = zgemm(dev, opa, opb, a if opa == 0 else a.conj().T, b if opb == 0 else b.conj().T, real)
    re, im = product(a, b, np.longdouble if real is np.float64 else np.float64)
    r4, i4 = product(a, b, real)
    assert norm(C.real - re, C.imag - im) <= norm(r4 - re, i4 - im)
    if kind == "rr":
        assert (C.imag == 0).all()
