"""What the phases' times of a result are times of."""
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,s", [(10, 5), (14, 7), (18, 8)])
def test_spectral_layout_is_device_time(dev, L, s):
    # a few kernels of these sizes, 5 us at most each with the gap in front of it;
    # not the host's look at the state's norm (a read-back and the launches after
    # it, 20 us or more).  The least of many calls, since a first kernel can wait.
    psi = ti.haar_state_torch(L, 3, dev)
    calls = [T.tnslq_spectral_sum(psi, L, list(range(s)), "purity", 4, 3) for _ in range(30)]
    least = min(c["t_layout_ms"] for c in calls)
    assert 0 < least <= 0.030
    for c in calls:
        assert c["t_layout_ms"] + c["t_matvec_ms"] + c["t_lanczos_ms"] <= c["t_total_ms"]


def test_quadrature_past_64_steps_costs_its_rotations(dev):
    # thousands of problems: the time is that of their rotations, whose number grows
    # with the cube of the steps; entries in a second register must not add to it
    psi = ti.haar_state_torch(13, 3, dev)
    run = {}
    for m in (64, 100):
        calls = [T.tnslq_logneg(psi, 13, [0, 1, 2, 3], [4, 5, 6, 7], 2048, m, precision="fp64", seed=1) for _ in range(4)]
        run[m] = min(c["t_total_ms"] - c["t_layout_ms"] - c["t_matvec_ms"] - c["t_lanczos_ms"] for c in calls)
    assert run[100] <= (100 / 64) ** 3 * run[64]
