"""Operands written in whole 16-byte units and LDS tiles: edges of the units
(2 to 8 terms), of the 64 x 32 tiles and of the regrouping's row order,
against the oracle; and the state check's sum off its strides."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import exact

pytestmark = pytest.mark.gpu

# the bars of the parity tests (norm-wise)
TOL = {"fp64": 1e-12, "fp32": 1e-6, "bf16x6": 1e-6, "bf16x3": 3e-5}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("L,a,b", [
    (13, [0, 1, 2, 3, 4, 5, 6], [7, 8, 9, 10, 11, 12]),   # d_B = 64: two tiles of b, no environment
    (13, [6, 7, 8, 9, 10, 11, 12], [0, 1, 2, 3, 4, 5]),   # psi's low bits in A
    (12, [0, 3, 6, 9], [1, 4, 7, 10]),                    # ... in the environment, everything interleaved
    (11, [1, 2], [3, 4]),                                 # d_A = 4: below a BF16 unit
    (11, [10], [0]),                                      # d_A = 2
    (12, [2, 3, 4, 5, 6], [7, 8]),                        # ... in E below B, d_B = 4
    (13, [1, 2, 3, 4], [5, 6, 7, 8, 9]),                  # roles exchanged
])
def test_matvec_at_unit_and_tile_edges(dev, prec, L, a, b):
    import torch
    psi = ti.haar_state(L, 2)
    X = ti.random_vectors(17, 1 << (len(a) + len(b)), seed=6)
    Y = T.tnslq_ptmatvec(torch.from_numpy(psi).to(dev), L, a, b, torch.from_numpy(X).to(dev), precision=prec)
    ref = exact.pt_matvec_explicit(exact.regroup(psi, L, a, b), X)
    assert np.linalg.norm(Y.cpu().numpy() - ref) <= TOL[prec] * np.linalg.norm(ref)


@pytest.mark.parametrize("dims", [(2, 3), (5, 7, 11), (3, 5, 7, 11, 13), (64, 64, 64, 5)])
@pytest.mark.parametrize("at", [0, 1, -1])
def test_state_check_sees_every_amplitude(dev, dims, at):
    # 1e-9 is the norm's tolerance in FP64: a state off by 1e-8 is refused, as
    # is one with a single non-finite amplitude, wherever it lies
    import torch
    psi = ti.haar_state_dims(list(dims), 1)
    run = lambda p: T.tnslq_logneg_dims(torch.from_numpy(p).to(dev), list(dims), [0], [1], 2, 1, precision="fp64")
    run(psi)
    bad = psi.copy()
    bad[at] = np.nan
    with pytest.raises(T.TnslqError) as e:
        run(bad)
    assert e.value.status == T.TNSLQ_E_NONFINITE
    bad = psi.copy()
    bad[at] += 1e-4 * (bad[at] / abs(bad[at]))
    if abs(np.vdot(bad, bad).real - 1) > 1e-8:
        with pytest.raises(T.TnslqError) as e:
            run(bad)
        assert e.value.status == T.TNSLQ_E_STATE
