"""Benchmark: seconds per +-1% logarithmic-negativity estimate of a 26-qubit
rho_AB (30-qubit Haar state, A = 4-16, B = 17-29, E = 0-3), on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]

One step is one whole estimate through the C ABI (tnslq_logneg): regrouping
psi into the contraction layouts, probe generation, the Lanczos loop with one
block matvec (both contractions) per step until the +-1% target of
``--stop-tol`` is met (at most ``--max-steps``), Gauss quadrature and the
Hutchinson statistics.  The state is generated on the device before timing.
Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "s per ±1% logneg estimate @26-qubit ρ_AB; ρ^T_B matvec GB/s or MFMA util"
# the matrix cores that the contractions of each precision run on (FP32 on the
# BF16 ones, in exact pieces)
PEAK_TFLOPS = {"bf16x3": 2500.0, "bf16x6": 2500.0, "fp32": 2500.0, "fp64": 78.6}
# matrix-core products per real product of the algorithm (4 per complex
# product): split BF16 takes 3 products of pieces per real product and 3 real
# products per complex one (9 / 4); BF16X6 6 products of pieces, 4 real
# products; FP32 6 products of pieces, 3 real products; FP64 3 real products
MFMA_PER_ALGO = {"bf16x3": 2.25, "bf16x6": 6.0, "fp32": 4.5, "fp64": 0.75}
# rocprofv3 counter summary of the split-BF16 contraction kernel at the default workload
COUNTERS = os.path.join(ROOT, "profiles", "gemm_bf16x3_haar30_counters.txt")


def read_counters(path=None):
    """key = value lines of a counter summary ('#' lines are comments)."""
    path = path or COUNTERS
    out = {}
    if not os.path.exists(path):
        return out
    with open(path) as f:
        for line in f:
            line = line.strip()
            if line and not line.startswith("#") and "=" in line:
                k, v = line.split("=", 1)
                out[k.strip()] = v.strip()
    return out


def kernel_source_sha256(files):
    import hashlib
    h = hashlib.sha256()
    for rel in files:
        with open(os.path.join(ROOT, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def counter_figures(workload_name, precision, kernel):
    """HBM bytes per launch (FETCH_SIZE and WRITE_SIZE passes, each scaled by the
    same counter's reading for a 1 GiB device copy) and the matrix-core busy
    fraction of `kernel`, from the committed counter summary; None when the
    summary is for another workload or precision, or the kernel's sources have
    changed since the counters were taken."""
    c = read_counters()
    if not c or workload_name != "haar30" or precision != "bf16x3":
        return None
    try:
        if kernel_source_sha256(c["kernel_sources"].split()) != c["kernel_source_sha256"]:
            return None
        return {"hbm_bytes": float(c[f"{kernel}_hbm_bytes"]),
                "mfma_busy_frac": float(c[f"{kernel}_mfma_busy_frac"]),
                "avg_clock_ghz": float(c[f"{kernel}_avg_clock_ghz"])}
    except (KeyError, ValueError, OSError):
        return None

EXTRA = {
    # 26-qubit Haar state with the same block structure (E = 4 qubits) but
    # d_A = d_B = 2^11: a quick proxy for kernel timing.
    "haar26": dict(n_qubits=26, a=tuple(range(4, 15)), b=tuple(range(15, 26)), n_probes=8, n_steps=50,
                   state="haar", dtype="c64", precision="bf16x3", reorth=False),
}


def finite_or_none(v):
    """The JSON line with every NaN or infinity as null (strict JSON has
    neither)."""
    import math
    if isinstance(v, float) and not math.isfinite(v):
        return None
    if isinstance(v, dict):
        return {k: finite_or_none(x) for k, x in v.items()}
    if isinstance(v, (list, tuple)):
        return [finite_or_none(x) for x in v]
    return v


def workload(name):
    import tnslq_inputs as ti
    if name in ti.WORKLOADS:
        w = ti.WORKLOADS[name]
        return dict(n_qubits=w.n_qubits, a=w.a, b=w.b, n_probes=w.n_probes, n_steps=w.n_steps, state=w.state,
                    dtype=w.dtype, precision=w.precision, reorth=w.reorth, depth=w.depth)
    return dict(EXTRA[name])


def make_state(w, seed, dev):
    import numpy as np
    import torch
    import tnslq_inputs as ti
    tdt = torch.complex64 if w["dtype"] == "c64" else torch.complex128
    if w["state"] == "haar":
        if w["n_qubits"] >= 24:
            return ti.haar_state_torch(w["n_qubits"], seed, dev, tdt)
        ndt = np.complex64 if w["dtype"] == "c64" else np.complex128
        return torch.from_numpy(ti.haar_state(w["n_qubits"], seed, ndt)).to(dev)
    return ti.brickwork_state_torch(w["n_qubits"], w.get("depth", 12), seed, dev, tdt)


def host_cpu():
    """The host's CPU model and logical CPU count."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return model, os.cpu_count()


def cpu_baseline(psi, w, m_used, budget_s=30.0):
    """Time the FP64 oracle on the host.  Where rho^{T_B} is small
    (d_A d_B <= 4096) the oracle runs in full: its exact eigensolve (Eq. 1)
    and its Algorithm 1 with the explicit matvec on the same K probes and
    steps; otherwise its lazy matvec (Sec. V Eq. 4) on a bounded sample of the
    same workload, scaled to one estimate."""
    import numpy as np
    from oracle import exact
    from threadpoolctl import threadpool_info
    L, a, b = w["n_qubits"], list(w["a"]), list(w["b"])
    threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    model, ncpu = host_cpu()
    if len(a) + len(b) <= 12:
        from oracle import slq
        psi_h = psi.cpu().numpy().astype(np.complex128)
        t0 = time.perf_counter()
        e_exact = exact.logneg_exact(exact.regroup(psi_h, L, a, b))
        t_eig = time.perf_counter() - t0
        t0 = time.perf_counter()
        o = slq.slq_logneg(psi_h, L, a, b, w["n_probes"], m_used, seed=0, reorth=bool(w["reorth"]))
        t_slq = time.perf_counter() - t0
        return {"value": t_slq, "unit": "s per estimate", "cores": threads, "kind": "oracle",
                "sample": f"full: Algorithm 1 with the explicit matvec, K = {w['n_probes']}, {m_used} fixed steps (no fit) "
                          f"({t_slq:.2f} s, E = {o['logneg']:.6f}); exact eigensolve of rho^T_B {t_eig:.2f} s "
                          f"(E = {e_exact:.6f}); host {model}, {ncpu} logical CPUs"}
    e = [q for q in range(L) if q not in a and q not in b]
    na, nb, ne = len(a), len(b), len(e)
    contiguous = e == list(range(ne)) and a == list(range(ne, ne + na)) and b == list(range(ne + na, L))
    K = w["n_probes"]
    if contiguous:
        # the environment is the leading qubits: slab c = 0 is psi[:d_A d_B]
        slab = psi[: 1 << (na + nb)].cpu().numpy().astype(np.complex128)
        P = slab.reshape(1 << na, 1 << nb, 1)
        n_slab = 1 << ne
        sample_desc = f"lazy FP64 matvec of 1 probe over 1 of {n_slab} environment slabs"
    else:
        P = exact.regroup(psi.cpu().numpy(), L, a, b)
        n_slab = 1
        sample_desc = "lazy FP64 matvec of 1 probe over the whole state"
    from tnslq_inputs import random_vectors
    x = random_vectors(1, P.shape[0] * P.shape[1], seed=0)
    t0 = time.perf_counter()
    exact.pt_matvec_lazy(P, x)
    t = time.perf_counter() - t0
    per_estimate = t * n_slab * K * m_used
    return {"value": per_estimate, "unit": "s per estimate (extrapolated)", "cores": threads, "kind": "oracle",
            "sample": f"{sample_desc}: {t:.2f} s, scaled x{n_slab} slabs x{K} probes x{m_used} Lanczos steps; "
                      f"host {model}, {ncpu} logical CPUs"}


def run_forms(args, w, psi, L, a, b, m, ws):
    """Each requested form on the same state and probes: seconds to the +-1%
    target, the estimate, and its difference from the FP64 form both at the
    stopping point and at a common step count (E_j from the quadrature values)."""
    import numpy as np
    import torch
    import paper_1809_01685_amd as T
    res = {}
    traj = {}
    for form in [f for f in args.forms.split(",") if f]:
        # "precision" or "precision:rule" (rule: fit or diff; default the run's)
        prec, _, rule = form.partition(":")
        rule = rule or args.stop_rule
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        if prec == "surrogate":
            from paper_1809_01685_amd import surrogate as S
            model = S.Model.load()
            r = S.surrogate_logneg(model, psi, L, a, b, w["n_probes"], m, tol=0.01, precision=w["precision"],
                                   seed=args.seed, stop_tol=args.stop_tol, workspace=ws, stop_rule=rule)
        else:
            r = T.tnslq_logneg(psi, L, a, b, w["n_probes"], m, reorth=w["reorth"], precision=prec, seed=args.seed,
                               stop_tol=args.stop_tol, workspace=ws if prec == w["precision"] else None,
                               stop_rule=rule)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        torch.cuda.empty_cache()
        entry = {"seconds": dt, "logneg": r["logneg"], "logneg_se": r["logneg_se"], "lanczos_err": r["lanczos_err"],
                 "lanczos_steps": r["steps_done"], "stop_rule": rule}
        if prec == "surrogate":
            entry.update({"mu": r["mu"], "sigma": r["sigma"], "e_early": r["e_early"],
                          "used_fallback": r["used_fallback"]})
        else:
            G = r["beta"][:, :1] ** 2 * r["F"][:, :r["steps_done"]]
            traj[form] = np.log2(G.mean(axis=0))
        res[form] = entry
        print(f"[bench] form {form}: {dt:.2f} s, E = {r['logneg']:.6f} after {r['steps_done']} steps",
              file=sys.stderr, flush=True)
    ref = next((f for f in traj if f.partition(":")[0] == "fp64"), None)
    if ref is not None:
        j = min(len(t) for t in traj.values())
        for form, t in traj.items():
            res[form]["logneg_at_common_step"] = float(t[j - 1])
            res[form]["error_vs_fp64_at_common_step"] = float(t[j - 1] - traj[ref][j - 1])
        res["common_step"] = j
        for form, e in res.items():
            if isinstance(e, dict):
                e["error_vs_fp64"] = float(e["logneg"] - res[ref]["logneg"])
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1)
    ap.add_argument("--warmup", type=int, default=0)
    ap.add_argument("--workload", default="haar30")
    ap.add_argument("--precision", default=None)
    ap.add_argument("--stop-tol", type=float, default=0.01)
    ap.add_argument("--stop-rule", default="fit", choices=["fit", "diff"],
                    help="fit: Algorithm 1's lanczos_estimate by the exponential fit of Sec. III; "
                         "diff: quadrature E_j with |E_j - E_{j-5}| as the Lanczos error")
    ap.add_argument("--check-steps", type=int, default=0, metavar="M",
                    help="also run M fixed steps on the same probes and report the estimate's error against "
                         "that run's value (post-hoc check of the +-tol target)")
    ap.add_argument("--save-trajectory", default="", metavar="NPZ",
                    help="with --check-steps: write that run's alpha, beta and quadrature values to NPZ")
    ap.add_argument("--max-steps", type=int, default=None)
    ap.add_argument("--probes", type=int, default=None)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--forms", default=None,
                    help="comma list of extra forms to time on the same state and probes "
                         "(fp64, fp32, bf16x3, bf16x6, surrogate); adds a 'forms' object with each form's "
                         "time, estimate and error against the FP64 form (default: the learned stop, "
                         "'surrogate', on the default haar30 run; '' for none)")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="first copy MIB MiB device-to-device (a known-size kernel for scaling HBM counters)")
    args = ap.parse_args()
    if args.forms is None:
        # the metric asks for the split-precision and the learned-stop forms
        # side by side; the default line carries the second as a form
        args.forms = "surrogate" if (args.workload == "haar30" and not args.max_steps and not args.check_steps) else ""
    if args.gpus != 1:
        print(json.dumps({"error": "this library runs on one GPU only; --gpus must be 1 "
                                   "(probe-sharded multi-GPU execution is designed but not built)"}))
        sys.exit(2)

    import torch
    import paper_1809_01685_amd as T

    dev = torch.device("cuda:0")
    if args.copy_calibration:
        src = torch.ones(args.copy_calibration << 20, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    w = workload(args.workload)
    if args.precision:
        w["precision"] = args.precision
    if args.probes:
        w["n_probes"] = args.probes
    m = args.max_steps or w["n_steps"]
    L, a, b = w["n_qubits"], list(w["a"]), list(w["b"])
    print(f"[bench] workload {args.workload}: L={L} |A|={len(a)} |B|={len(b)} K={w['n_probes']} m<={m} "
          f"{w['precision']} stop_tol={args.stop_tol}", file=sys.stderr, flush=True)
    psi = make_state(w, args.seed, dev)
    dtc = T.TNSLQ_C64 if psi.dtype == torch.complex64 else T.TNSLQ_C128
    opts = T.make_options(w["n_probes"], max(m, args.check_steps), w["reorth"], w["precision"], args.seed, 0,
                          args.stop_tol, args.stop_rule)
    nbytes = T.tnslq_workspace_bytes(dtc, L, a, b, opts)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    print(f"[bench] state ready, workspace {nbytes / 2**30:.2f} GiB", file=sys.stderr, flush=True)

    def step():
        return T.tnslq_logneg(psi, L, a, b, w["n_probes"], m, reorth=w["reorth"], precision=w["precision"],
                              seed=args.seed, stop_tol=args.stop_tol, workspace=ws, want_arrays=False,
                              stop_rule=args.stop_rule)

    for i in range(args.warmup):
        step()
        print(f"[bench] warmup {i + 1}/{args.warmup} done", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    results = []
    for i in range(args.steps):
        results.append(step())
        print(f"[bench] step {i + 1}/{args.steps}: E = {results[-1]['logneg']:.6f} +- {results[-1]['logneg_se']:.2e}"
              f" after {results[-1]['steps_done']} Lanczos steps, {results[-1]['t_total_ms'] / 1e3:.2f} s",
              file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = 1e3 * elapsed / args.steps

    last = results[-1]
    d_a, d_b = 1 << len(a), 1 << len(b)
    d_min = min(d_a, d_b)
    D = 1 << L
    kc_launch = max(1, w["n_probes"] * last["steps_done"] // max(1, last["n_contract_launches"]))
    flops_per_launch = 8.0 * D * d_min * kc_launch           # one contraction over kc probes
    t1 = last["t_contract1_ms"] / max(1, last["n_contract_launches"])
    t2 = last["t_contract2_ms"] / max(1, last["n_contract_launches"])
    dom, tdom = ("contraction2", t2) if t2 >= t1 else ("contraction1", t1)
    achieved = flops_per_launch / (tdom * 1e-3) / 1e12
    peak = PEAK_TFLOPS[w["precision"]]
    counters = counter_figures(args.workload, w["precision"], dom)
    out = {
        "metric": METRIC,
        "value": ms_per_step / 1e3,
        "unit": "s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"bf16x3": "bf16 (hi+lo split, f32 acc) + f64 Lanczos",
                  "bf16x6": "bf16 (3-piece split, f32 acc) + f64 Lanczos",
                  "fp32": "f32 + f64 Lanczos", "fp64": "f64"}[w["precision"]],
        "data": "synthetic",
        "config": {"workload": f"{args.workload}: {L}-qubit {w['state']} state {w['dtype']}, A={a[0]}-{a[-1]}, "
                               f"B={b[0]}-{b[-1]}, {len(a) + len(b)}-qubit rho_AB, K={w['n_probes']} probes, "
                               f"<= {m} Lanczos steps, stop at +-{args.stop_tol * 100:g}% "
                               f"({'exponential-fit' if args.stop_rule == 'fit' else 'step-difference'} rule)",
                   "precision": w["precision"], "reorth": bool(w["reorth"])},
        "result": {"logneg": last["logneg"], "logneg_se": last["logneg_se"], "lanczos_err": last["lanczos_err"],
                   "lanczos_steps": last["steps_done"], "stop_rule": args.stop_rule,
                   "t_layout_ms": last["t_layout_ms"], "t_matvec_ms": last["t_matvec_ms"],
                   "t_lanczos_ms": last["t_lanczos_ms"]},
        "roofline": {"bound": "mfma", "kernel": dom, "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                     "frac": achieved / peak, "mfma_issue_frac": achieved * MFMA_PER_ALGO[w["precision"]] / peak,
                     "flops_per_launch": flops_per_launch, "avg_launch_ms": tdom,
                     "traffic": counters["hbm_bytes"] if counters else None},
    }
    if counters:
        out["roofline"]["counters"] = {"source": os.path.relpath(COUNTERS, ROOT),
                                       "mfma_busy_frac": counters["mfma_busy_frac"],
                                       "avg_clock_ghz": counters["avg_clock_ghz"]}
    if args.check_steps:
        # the plain M-step estimate (Gauss quadrature of T_M) on the same probes
        ref = T.tnslq_logneg(psi, L, a, b, w["n_probes"], args.check_steps, reorth=w["reorth"],
                             precision=w["precision"], seed=args.seed, stop_tol=0.0, workspace=ws,
                             want_arrays=bool(args.save_trajectory), stop_rule="diff")
        if args.save_trajectory:
            import numpy as np
            np.savez(args.save_trajectory, alpha=ref["alpha"], beta=ref["beta"], F=ref["F"])
        out["accuracy_check"] = {"reference_steps": args.check_steps, "reference_logneg": ref["logneg"],
                                 "error": last["logneg"] - ref["logneg"],
                                 "target": args.stop_tol * max(abs(ref["logneg"]), 1.0)}
        print(f"[bench] check: {args.check_steps}-step value {ref['logneg']:.6f}, error of the estimate "
              f"{last['logneg'] - ref['logneg']:+.4f}", file=sys.stderr, flush=True)
    if args.forms:
        out["forms"] = run_forms(args, w, psi, L, a, b, m, ws)
    if not args.no_cpu_baseline:
        print("[bench] timing the oracle sample on the host", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(psi, w, last["steps_done"])
    print(json.dumps(finite_or_none(out), allow_nan=False), flush=True)


if __name__ == "__main__":
    main()
