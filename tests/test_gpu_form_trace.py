"""FP32 explicit operator: the trace of rho_AB, summed from squares, leans to no side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [18, 20])   # traced side 256 and 1024
def test_trace_of_formed_operator_is_unbiased(L):
    # <z, rho z> of one Lanczos step, FP32 against FP64 on the same complex64
    # state.  The error of a diagonal element is a few roundings of its sum, at
    # most 1.2e-7 of it in the standard deviation; the mean over 1024 elements
    # and 4 states has 1.9e-9.  Five of those.
    import paper_1809_01685_amd as T
    a, b, n = list(range(5)), list(range(5, 10)), 1024
    means = []
    for s in range(4):
        g = torch.Generator(device="cuda")
        g.manual_seed(100 + s)
        x = torch.randn(1 << L, dtype=torch.complex128, device="cuda", generator=g)
        psi = (x / torch.linalg.vector_norm(x)).to(torch.complex64)
        al = {p: T.tnslq_logneg(psi, L, a, b, 256, 1, precision=p, seed=s, operator="explicit")["alpha"]
              for p in ("fp32", "fp64")}
        means.append(((al["fp32"] - al["fp64"]) * n).mean())
    assert abs(np.mean(means)) <= 1e-8, means


@pytest.mark.parametrize("kind", ["complex", "positive"])
@pytest.mark.parametrize("L", [14, 16])   # traced side 256 and 1024
def test_trace_of_small_formed_operator_is_unbiased(L, kind):
    # 64 elements: 1.5e-8 in the standard deviation of one state's mean, 2.4e-9
    # over 40 states.  Five of those.
    import paper_1809_01685_amd as T
    a, b, n = [0, 1, 2], [3, 4, 5], 64
    means = []
    for s in range(40):
        g = torch.Generator(device="cuda")
        g.manual_seed(500 + s)
        if kind == "complex":
            x = torch.randn(1 << L, dtype=torch.complex128, device="cuda", generator=g)
        else:
            x = torch.rand(1 << L, dtype=torch.float64, device="cuda", generator=g) + 0.5 + 0j
        psi = (x / torch.linalg.vector_norm(x)).to(torch.complex64)
        al = {p: T.tnslq_logneg(psi, L, a, b, 64, 1, precision=p, seed=s, operator="explicit")["alpha"]
              for p in ("fp32", "fp64")}
        means.append(((al["fp32"] - al["fp64"]) * n).mean())
    assert abs(np.mean(means)) <= 1.2e-8, np.mean(means)
