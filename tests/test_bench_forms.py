"""bench.py times several precisions of one workload: each has the workspace that
its own plan asks for, which in FP32 is not the largest of them (host only)."""
import argparse
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import paper_1809_01685_amd as T  # noqa: E402
import tnslq_inputs as ti  # noqa: E402


@pytest.mark.parametrize("workload", ["haar10", "haar20", "brick24", "haar30"])
def test_every_form_has_its_workspace(workload, monkeypatch):
    import torch
    wl = ti.WORKLOADS[workload]
    w = {"n_probes": wl.n_probes, "reorth": wl.reorth, "precision": wl.precision}
    L, a, b, m = wl.n_qubits, list(wl.a), list(wl.b), wl.n_steps

    def need(prec):
        return T.tnslq_workspace_bytes(T.TNSLQ_C64, L, a, b,
                                       T.make_options(wl.n_probes, m, wl.reorth, prec, 0, 0, 0.01, "fit"))

    class Workspace:
        def __init__(self, n):
            self.n = n

        def numel(self):
            return self.n

    seen = []

    def logneg(psi, L, a, b, K, m, precision, workspace, **kw):
        assert workspace is None or workspace.numel() >= need(precision), precision
        seen.append(precision)
        return {"logneg": 1.0, "logneg_se": 0.0, "lanczos_err": 0.0, "steps_done": 1,
                "beta": np.ones((K, 2)), "F": np.ones((K, 1))}

    monkeypatch.setattr(T, "tnslq_logneg", logneg)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: None)
    args = argparse.Namespace(forms="fp64:fit,fp32:fit,bf16x3:fit,bf16x6:fit", stop_rule="fit", stop_tol=0.01, seed=0)
    bench.run_forms(args, w, None, L, a, b, m, Workspace(need(wl.precision)))
    assert seen == ["fp64", "fp32", "bf16x3", "bf16x6"]
