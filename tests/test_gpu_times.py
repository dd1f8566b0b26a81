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
