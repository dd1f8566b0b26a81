"""Bias gradients as row sums inside the weight-gradient products: batches at
the edges of a lane's 8 terms, a step's 32 and the four waves' 128, against
the oracle.  Tolerance: 1e-5 norm-wise per block, as the gradient's own test
(FP32 against FP64 sums of at most a few hundred terms)."""
import numpy as np
import pytest

import paper_1809_01685_amd as T
import tnslq_inputs as ti
from oracle import mlp

pytestmark = pytest.mark.gpu

BIASES = [("b1", 4864, 5120), ("b2", 70656, 70912), ("b3", 71424, 71426)]


@pytest.mark.parametrize("B", [1, 8, 9, 31, 33, 127, 129, 300])
def test_bias_gradients(dev, B):
    import torch
    rng = np.random.default_rng(B)
    th = ti.mlp_init_params(5)
    x = (rng.standard_normal((B, 19)) * 3 + 1).astype(np.float32)
    r = rng.standard_normal(B).astype(np.float32)
    norm = np.concatenate([rng.standard_normal(19), rng.uniform(0.5, 2.0, 19)]).astype(np.float32)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    _, grad = T.tnslq_mlp_loss_grad(up(th), up(norm), up(x), up(r))
    grad = grad.cpu().numpy().astype(np.float64)
    xh = mlp.standardise(x.astype(np.float64), norm[:19].astype(np.float64), norm[19:].astype(np.float64))
    _, want, _ = mlp.loss_and_grad(th.astype(np.float64), xh, r.astype(np.float64))
    for name, a, b in BIASES:
        assert np.linalg.norm(grad[a:b] - want[a:b]) <= 1e-5 * max(np.linalg.norm(want[a:b]), 1e-30), name
