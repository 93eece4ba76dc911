#!/usr/bin/env python3
"""Benchmark: policy x scenario reserve valuations per second, exact FP64.

Workload (one step = one full pass of the hot path): 10,000 mixed policies
(40 % single-life annuities, 20 % joint-life annuities, 20 % term
assurances, 20 % endowments; ages 20-85, remaining terms 60-600 months) x
1,000 Vasicek inner scenarios, FP64 backward recurrence to t = 0 for every
policy x scenario, per-policy reserves written to HBM, portfolio totals per
scenario and the 1-in-200 tail statistic.  Inputs are seeded synthetic data
resident in device memory before timing starts.

Prints one JSON line.  Also measured: the recurrence kernel's duration with
HIP events around every launch of a second timed region (roofline), the
same workload's single-scenario and 60-node variants, and the CPU oracle on a
bounded sample of the workload on this host's cores.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

FP64_PEAK_TFLOPS = 78.6        # MI355X FP64 vector, FMA = 2 flops
FP64_ISSUE_PEAK = 39.3e12      # 256 CU x 4 SIMD x 16 lanes x 2.4 GHz, one op per lane-cycle


def scenario_step_work(pf, node=0, node_step=12):
    """Algorithmic FP64 flops and VALU ops per scenario of one pass, summed over
    policies: the per-scenario arithmetic of the zero-reserve-reduced
    recurrence (per-policy work shared by all scenarios is not counted)."""
    import synth
    S = np.maximum(pf.term_m.astype(np.int64) - node * node_step, 0)
    prod = pf.product
    prem = pf.premium > 0
    arrears = pf.timing == synth.ARREARS
    flops = np.zeros(pf.n)
    ops = np.zeros(pf.n)
    # single-state recurrences: r = a0 + v (p r + c)
    single = np.isin(prod, (synth.SL_ANN, synth.JL_ANN, synth.TERM, synth.ENDOW, synth.ENDOW_ASSUR,
                            synth.CF_TABLE))
    c_nonzero = ((np.isin(prod, (synth.SL_ANN, synth.JL_ANN)) & arrears) |
                 np.isin(prod, (synth.TERM, synth.ENDOW_ASSUR, synth.CF_TABLE)))
    a0_nonzero = prem | (np.isin(prod, (synth.SL_ANN, synth.JL_ANN)) & ~arrears)
    flops[single] = (np.where(c_nonzero, 2, 1) + np.where(a0_nonzero, 2, 1))[single]
    ops[single] = 2
    rev = prod == synth.REV_ANN
    flops[rev] = (4 + np.where(prem, 2, 1) + 2 + np.where(~arrears, 2, 1))[rev]
    ops[rev] = 5
    ls = prod == synth.LS_ANN
    flops[ls] = (6 + np.where(prem | ~arrears, 2, 1) + 2 * (2 + np.where(~arrears, 2, 1)))[ls]
    ops[ls] = 8
    # two-life endowment / first-death assurance: scalar chains; second death: 3-vector
    jl_end, jl_a1, jl_a2 = prod == synth.JL_ENDOW, prod == synth.JL_ASSUR1, prod == synth.JL_ASSUR2
    flops[jl_end] = (1 + np.where(prem, 2, 1))[jl_end]
    flops[jl_a1] = (2 + np.where(prem, 2, 1))[jl_a1]
    ops[jl_end | jl_a1] = 2
    flops[jl_a2] = (6 + np.where(prem, 2, 1) + 2 * 3)[jl_a2]
    ops[jl_a2] = 8
    return float((flops * S).sum()), float((ops * S).sum()), int((S > 0).sum()), int(S.sum())


CSRC = os.path.join(ROOT, "paper_1401_1757_amd", "csrc")
# Committed FETCH_SIZE / WRITE_SIZE counters of the C3 launch, and the kernel
# sources that they hold for: the recurrence kernel, a run by cash flows.
TRAFFIC = {False: (os.path.join(ROOT, "profiles", "k_recurrence_c3_10k_policies_1000_scenarios_traffic.json"),
                   ("rr_recurrence.h", "rr_internal.h")),
           True: (os.path.join(ROOT, "profiles", "k_reserve_mm_c3_10k_policies_1000_scenarios_traffic.json"),
                  ("rr_flows.h", "rr_flows.hip", "rr_reserve_mm.hip", "rr_recurrence.h", "rr_internal.h"))}


def source_sha(by_flows):
    import hashlib
    h = hashlib.sha256()
    for src in TRAFFIC[by_flows][1]:
        with open(os.path.join(CSRC, src), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def measured_traffic(k, j, wg, ring=0):
    """HBM bytes per launch (k = 0: per run by cash flows, its kernels together)
    from the committed counters, if they were taken on these kernel sources and
    this launch shape."""
    by_flows = k == 0
    try:
        with open(TRAFFIC[by_flows][0]) as f:
            t = json.load(f)
        sha = source_sha(by_flows)
    except OSError:
        return None
    launch = dict(t.get("launch", {}))
    launch.setdefault("curve_ring", 0)
    if t.get("source_sha256") != sha or (not by_flows and launch != {"block_k": k, "block_j": j, "wg_per_cu": wg,
                                                                     "curve_ring": ring}):
        return None
    return float(t["traffic_bytes_per_launch"])


def algorithmic_bytes(b, pf):
    """Bytes one launch must move: every scenario curve once, the policy
    records once and every reserve written once, plus the per-tile partial
    totals."""
    curves = b.n_scen * b.n_steps * 8
    policies = pf.n * (6 * 4 + 6 * 8)
    r0 = pf.n * b.n_scen * 8
    partials = ((pf.n + 63) // 64) * b.n_scen * 8
    return float(curves + policies + r0 + partials)


def timed_steps(fn, steps, sync):
    sync()
    t0 = time.perf_counter()
    for _ in range(steps):
        fn()
    sync()
    return time.perf_counter() - t0


def cpu_model() -> str:
    """The host CPU's model name (lscpu's "Model name", from /proc/cpuinfo)."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.lower().startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_share() -> int:
    """Threads for the CPU leg: the CPU share this process is given
    (OMP_NUM_THREADS, where it is set per GPU), else every core."""
    val = os.environ.get("OMP_NUM_THREADS", "").strip()
    if val.isdigit() and int(val) > 0:
        return int(val)
    return os.cpu_count() or 1


def cpu_baseline(w, reps=7, seconds_per_run=1.2):
    """The oracle's reduced mode (zero-reserve states removed, the same
    per-product recurrences the GPU runs; pinned to the dense mode) on a
    bounded sample of the workload -- the whole portfolio over the first
    scenarios -- with the process's CPU share and with one core, minimum and
    median of `reps` runs each; the dense general form once, for
    information."""
    import oracle
    b, pf = w.basis, w.portfolio
    nproc = os.cpu_count() or 1
    share = cpu_share()

    def sample(threads):
        t0 = time.perf_counter()
        oracle.reserves_reduced(b, pf, 0, 1, 0, 1, n_threads=threads, want_r=False)
        per_scen = time.perf_counter() - t0
        n_scen = int(max(1, min(b.n_scen, round(seconds_per_run / max(per_scen, 1e-6)))))
        ts = []
        for _ in range(reps):
            t0 = time.perf_counter()
            oracle.reserves_reduced(b, pf, 0, 1, 0, n_scen, n_threads=threads, want_r=False)
            ts.append(time.perf_counter() - t0)
        ts = np.array(ts)
        vals = pf.n * n_scen / ts
        return {"threads": threads, "scenarios": n_scen, "valuations_per_s_best": float(vals.max()),
                "valuations_per_s_median": float(np.median(vals)), "seconds_min": float(ts.min()),
                "seconds_median": float(np.median(ts))}

    multi = sample(share)
    single = sample(1)
    t0 = time.perf_counter()
    n_dense = max(1, min(b.n_scen, multi["scenarios"] // 8))
    oracle.reserves(b, pf, 0, 1, 0, n_dense, want_gross=False, n_threads=share)
    dense_val = pf.n * n_dense / (time.perf_counter() - t0)
    return {"value": multi["valuations_per_s_median"], "unit": "valuations/s", "cores": share,
            "kind": "oracle",
            "sample": f"all {pf.n} policies x first {multi['scenarios']} scenarios of the workload, "
                      f"oracle reduced mode (zero-reserve states removed), {share} OpenMP threads, "
                      f"median of {reps} runs; 1 core: all policies x first {single['scenarios']} "
                      f"scenarios",
            "nproc": nproc, "cpu_model": cpu_model(),
            "threads_note": "the process's CPU share (OMP_NUM_THREADS), not every core nproc shows",
            "share": multi, "one_core": single,
            "one_core_valuations_per_s": single["valuations_per_s_median"],
            "dense_general_form_valuations_per_s": dense_val,
            "dense_sample_scenarios": n_dense}


SURROGATE_TRAIN = dict(seed=1005, n=5000, n_nodes=20, n_scen=100)
SURROGATE_FIT = dict(epochs=24, batch=8192, lr=2e-3, lr_final=1e-5, holdout=0.01, seed=11)
MLP_FLOPS_PER_ROW = 2 * (17 * 256 + 256 * 256 + 256)   # algorithmic: 17 inputs, two 256-wide layers, head


def surrogate_leg(rr, synth, ctx, w, exact_totals, n_val, exact_ms, steps, sync, profile_only=False,
                  epochs=0):
    """Train the MLP surrogate on GPU-generated exact samples, then time its
    inference over the same workload (same outputs as the exact step)."""
    tw = synth.surrogate_training_workload(**SURROGATE_TRAIN)
    ctx.basis_upload(tw.basis.q, tw.basis.v, tw.basis.shock)
    ctx.portfolio_upload(tw.portfolio)
    t0 = time.perf_counter()
    fit = dict(SURROGATE_FIT)
    if epochs:
        fit["epochs"] = epochs
    rep = ctx.surrogate_train(node_step=0, **fit)
    train_s = time.perf_counter() - t0
    b, pf = w.basis, w.portfolio
    ctx.basis_upload(b.q, b.v, b.shock)
    ctx.portfolio_upload(pf)
    out = ctx.alloc_outputs(1, b.n_scen, stats=True)
    ctx.surrogate_infer(0, 1, 0, b.n_scen, 12, out)
    sync()
    counts = out.pop("report")
    step = lambda: ctx.surrogate_infer(0, 1, 0, b.n_scen, 12, out, report=False)
    for _ in range(3):
        step()
    elapsed = timed_steps(step, steps, sync)
    if profile_only:
        return {"ms_per_step": 1e3 * elapsed / steps}
    ctx.set_option(rr.OPT_KERNEL_TIMING, 1)
    ctx.kernel_times()
    timed_steps(step, steps, sync)
    kms = float(np.mean(ctx.kernel_times()))
    ctx.set_option(rr.OPT_KERNEL_TIMING, 0)
    sur_totals = out["totals"].cpu().numpy()[0]
    ms = 1e3 * elapsed / steps
    flops = MLP_FLOPS_PER_ROW * counts["n_in_range"]
    k = int(np.ceil(0.005 * b.n_scen))
    q = lambda x: np.sort(x)[::-1][k - 1]
    return {
        "valuations_per_s": n_val / (elapsed / steps),
        "ms_per_step": ms,
        "speedup_vs_exact": exact_ms / ms,
        "dtype": "bf16 (fp32 accumulate), fp64 fallback",
        "rows_network": counts["n_in_range"], "rows_fallback": counts["n_fallback"],
        "portfolio_reserve_rel_err": float(abs(sur_totals.mean() - exact_totals.mean()) /
                                           abs(exact_totals.mean())),
        "per_scenario_rms_rel_err": float(np.sqrt(np.mean(((sur_totals - exact_totals) / exact_totals) ** 2))),
        "tail_rel_err": float((q(sur_totals) - q(exact_totals)) / q(exact_totals)),
        "error_reference": "exact FP64 GPU recurrence of the same step",
        "roofline": {"bound": "mfma", "kernel": "k_infer", "kernel_ms": kms,
                     "achieved": flops / (kms * 1e-3) / 1e12, "peak": 2500.0, "unit": "TFLOP/s",
                     "frac": flops / (kms * 1e-3) / 2.5e15,
                     "algorithmic_flops_per_launch": float(flops)},
        "train": {"workload": tw.name, "samples": rep["n_samples"], "steps": rep["steps"],
                  "seconds": train_s, "data_ms": rep["data_ms"], "train_ms": rep["train_ms"],
                  "first_loss": rep["first_loss"], "final_loss": rep["final_loss"],
                  "holdout_loss": rep["holdout_loss"]},
    }


def c2_legs(rr, synth, ctx, sync, steps=20, path_only=False):
    """C2 (100,000 mixed policies, one flat scenario): r0 and totals per call
    (latency-bound), then path mode (the state-0 reserve at every step of
    every policy), bound by the HBM writes of the path."""
    w2 = synth.config_c2()
    ctx.basis_upload(w2.basis.q, w2.basis.v)
    ctx.portfolio_upload(w2.portfolio)
    out = {}
    if not path_only:
        o2 = ctx.alloc_outputs(1, 1)
        f2 = lambda: ctx.reserve_recurrence(0, 1, 0, 1, 12, o2)
        for _ in range(3):
            f2()
        e2 = timed_steps(f2, steps, sync)
        out["C2_single_scenario"] = {"valuations_per_s": w2.portfolio.n / (e2 / steps),
                                     "ms_per_step": 1e3 * e2 / steps, "policies": w2.portfolio.n}
    po = ctx.alloc_outputs(1, 1, r0=False, totals=False, path_node=0)
    fp = lambda: ctx.reserve_recurrence(0, 1, 0, 1, 12, po)
    for _ in range(3):
        fp()
    ep = timed_steps(fp, steps, sync)
    ctx.set_option(rr.OPT_KERNEL_TIMING, 1)
    ctx.kernel_times()
    timed_steps(fp, steps, sync)
    kp = float(np.mean(ctx.kernel_times()))
    ctx.set_option(rr.OPT_KERNEL_TIMING, 0)
    path_bytes = po["path"].numel() * 8
    out["C2_path_mode"] = {"ms_per_step": 1e3 * ep / steps, "kernel_ms": kp,
                           "path_bytes": path_bytes,
                           "kernel_write_GBps": path_bytes / (kp * 1e-3) / 1e9,
                           "frac_hbm_peak": path_bytes / (kp * 1e-3) / 8e12,
                           "policy_steps": int(po["path"].numel())}
    return out


def generated_scenarios_leg(rr, synth, sync, steps=20):
    """C3 with its 1,000 Vasicek scenarios generated on the device each step
    (a fresh Philox key per step): generation alone, and generation plus the
    recurrence, totals and tail statistic."""
    w = synth.config_c3()
    b, pf = w.basis, w.portfolio
    a, mean, sig, dt = synth.VAS_A, synth.VAS_B, synth.VAS_SIGMA, 1.0 / 12.0
    ctx = rr.Context(0)
    try:
        ctx.basis_generate_vasicek(b.q, b.n_scen, b.n_steps, [synth.VAS_R0], a, mean, sig, dt, (1, 0))
        ctx.portfolio_upload(pf)
        o = ctx.alloc_outputs(1, b.n_scen, stats=True)
        key = [0]

        def gen():
            key[0] += 1
            ctx.curves_generate_vasicek([synth.VAS_R0], a, mean, sig, dt, (1, key[0]))

        def full():
            gen()
            ctx.reserve_recurrence(0, 1, 0, b.n_scen, 12, o)

        for _ in range(3):
            full()
        sync()
        eg = timed_steps(gen, steps, sync)
        ef = timed_steps(full, steps, sync)
        _, _, live, _ = scenario_step_work(pf)
        return {"workload": w.name + ", scenarios generated on the device each step",
                "generation_ms": 1e3 * eg / steps, "ms_per_step": 1e3 * ef / steps,
                "valuations_per_s": live * b.n_scen / (ef / steps),
                "generated_values": b.n_scen * b.n_steps}
    finally:
        ctx.close()


def node_means_leg(rr, synth, sync, steps=10):
    """C4 (60 annual nodes x 500 inner scenarios): the expected portfolio
    reserve per node three ways: all inner scenarios (exact, the mean of the
    scenario totals), the mean discount curve (exact by linearity, one
    recurrence per node and policy), and the node-level surrogate (trained
    on the node training workload)."""
    w = synth.config_c4()
    b, pf = w.basis, w.portfolio
    K, S = b.n_nodes, b.n_scen
    ctx = rr.Context(0)
    try:
        tw = synth.node_training_workload()
        ctx.basis_upload(tw.basis.q, tw.basis.v, tw.basis.shock)
        ctx.portfolio_upload(tw.portfolio)
        t0 = time.perf_counter()
        rep = ctx.node_surrogate_train(node_step=tw.node_step_m, epochs=60, batch=4096, lr=2e-3,
                                       lr_final=1e-5, holdout=0.02, seed=3)
        sync()
        train_s = time.perf_counter() - t0
        ctx.basis_upload(b.q, b.v, b.shock)
        ctx.portfolio_upload(pf)
        ex = ctx.alloc_outputs(K, S, r0=False, stats=True)
        f_all = lambda: ctx.reserve_recurrence(0, K, 0, S, 12, ex)
        f_mean = lambda: ctx.node_expected_reserves(0, K, 0, S, 12, r0=False)
        f_sur = lambda: ctx.node_surrogate_infer(0, K, 0, S, 12, r0=False, report=False)
        res = {}
        for name, fn in (("all_scenarios", f_all), ("mean_curve", f_mean), ("surrogate", f_sur)):
            fn()
            fn()   # (captured)
            sync()
            res[name] = 1e3 * timed_steps(fn, steps, sync) / steps
        exact = ex["stats"].cpu().numpy()[:, 0]
        mc = f_mean()["totals"].cpu().numpy()
        so = ctx.node_surrogate_infer(0, K, 0, S, 12, r0=False)
        su = so["totals"].cpu().numpy()
        live = np.abs(exact) > 0
        rel = lambda x: float(np.max(np.abs(x[live] - exact[live]) / np.abs(exact[live])))
        return {"workload": w.name + ": expected portfolio reserve per node",
                "ms_all_scenarios": res["all_scenarios"], "ms_mean_curve": res["mean_curve"],
                "ms_surrogate": res["surrogate"],
                "max_rel_err_mean_curve": rel(mc), "max_rel_err_surrogate": rel(su),
                "surrogate_rows": so["report"],
                "surrogate_train_s": train_s, "surrogate_train_samples": rep["n_samples"],
                "reference": "mean over the 500 scenarios of the exact portfolio totals"}
    finally:
        ctx.close()


def representative_leg(rr, synth, sync, steps=5):
    """The representative annuity portfolio (Sec. 5.3, Table 2): 500,000
    annuities x 1,000 Vasicek scenarios over the 756 monthly steps to the
    limiting age, node 0, portfolio totals and the tail statistic."""
    w = synth.config_rep()
    b, pf = w.basis, w.portfolio
    ctx = rr.Context(0)
    try:
        ctx.basis_upload(b.q, b.v, b.shock)
        ctx.portfolio_upload(pf)
        o = ctx.alloc_outputs(1, b.n_scen, r0=False, stats=True)
        f = lambda: ctx.reserve_recurrence(0, 1, 0, b.n_scen, 12, o)
        t0 = time.perf_counter()
        f()
        sync()
        first = time.perf_counter() - t0
        f()
        e = timed_steps(f, steps, sync)
        ctx.set_option(rr.OPT_KERNEL_TIMING, 1)
        ctx.kernel_times()
        timed_steps(f, steps, sync)
        kms = float(np.mean(ctx.kernel_times()))
        ctx.set_option(rr.OPT_KERNEL_TIMING, 0)
        flops, ops, live, vsteps = scenario_step_work(pf)
        ms = 1e3 * e / steps
        chains = ctx.get_option(rr.OPT_LAST_K) > 0   # else summed cash flows: other work
        achieved = flops * b.n_scen / (kms * 1e-3) / 1e12 if chains else None
        return {"workload": w.name, "policies": pf.n, "scenarios": b.n_scen,
                "ms_per_step": ms, "kernel_ms": kms,
                "kernel_tflops": achieved, "kernel_frac_fp64_peak": achieved / FP64_PEAK_TFLOPS if chains else None,
                "kernel_issue_frac": ops * b.n_scen / (kms * 1e-3) / FP64_ISSUE_PEAK if chains else None,
                # totals by summed cash flows form no reserve per policy and scenario
                "valuations_per_s": live * b.n_scen / (e / steps) if chains else None,
                "valuation_steps_per_s": vsteps * b.n_scen / (e / steps) if chains else None,
                "scenario_totals_per_s": b.n_scen / (e / steps), "policies_in_a_total": live,
                "escalating": int((pf.escalation > 0).sum()), "annual": int(pf.annual.sum()),
                "launch": {"block_k": ctx.get_option(rr.OPT_LAST_K),
                           "block_j": ctx.get_option(rr.OPT_LAST_J),
                           "wg_per_cu": ctx.get_option(rr.OPT_LAST_WG),
                           "curve_ring": ctx.get_option(rr.OPT_LAST_RING),
                           "windows": ctx.get_option(rr.OPT_LAST_WINDOWS)},
                "first_call_s": first,
                "paper_context": "the paper estimates 5.7 s wall per scenario for this portfolio "
                                 "on a 2-core laptop CPU (Sec. 5.3); here ms_per_step covers "
                                 "all 1,000 scenarios"}
    finally:
        ctx.close()


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-secondary", action="store_true", help="skip the C2 / C4 variants")
    ap.add_argument("--no-surrogate", action="store_true", help="skip training and timing the surrogate")
    ap.add_argument("--surrogate-only", action="store_true",
                    help="only the surrogate's timed inference region (for profiling)")
    ap.add_argument("--calib-copy", action="store_true",
                    help="only run a plain 1 GiB device copy (traffic counter calibration)")
    ap.add_argument("--kernel-only", action="store_true",
                    help="only the timed region of the headline workload (for profiling)")
    ap.add_argument("--node-means-only", action="store_true",
                    help="only the C4 expected-reserve-per-node leg")
    ap.add_argument("--generated-only", action="store_true",
                    help="only the device-generated-scenario leg (for profiling)")
    ap.add_argument("--c2-only", action="store_true",
                    help="only the C2 legs (one scenario: r0 mode, then path mode)")
    ap.add_argument("--c2-path-only", action="store_true", help="only the C2 path-mode leg")
    ap.add_argument("--representative-only", action="store_true",
                    help="only the representative 500,000-annuity portfolio leg (for profiling)")
    ap.add_argument("--block-k", type=int, default=0, help="pin scenarios per lane (0 = autotune)")
    ap.add_argument("--wg", type=int, default=0, help="pin workgroups per CU (0 = autotune)")
    ap.add_argument("--block-j", type=int, default=0, help="pin policies per lane (0 = autotune)")
    ap.add_argument("--lane-spread", type=int, default=1,
                    help="1: deal tile lanes over the LDS banks (default), 0: sorted lane order")
    ap.add_argument("--curve-share", type=int, default=-1,
                    help="2: workgroups take windows of items of one scenario block together, "
                         "1: the same order taken item by item, 0: plain queues, "
                         "-1: 2 or 1 as the autotuner finds (default)")
    ap.add_argument("--ring", type=int, default=0,
                    help="curve ring for level portfolios: -1 autotune, 0 off (default), 1 on")
    ap.add_argument("--term-bucket", type=int, default=0, help="months per term bucket (0 = default)")
    ap.add_argument("--surrogate-epochs", type=int, default=0,
                    help="epochs of the surrogate training (0 = the default fit)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; --gpus must be 1",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU available"}))
        sys.exit(1)
    if args.calib_copy:
        a = torch.empty(1 << 27, dtype=torch.float64, device="cuda").fill_(1.0)
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": a.numel() * 8}))
        return

    import paper_1401_1757_amd as rr
    import synth

    sync = torch.cuda.synchronize
    if args.representative_only:
        print(json.dumps(representative_leg(rr, synth, sync, steps=args.steps)))
        return
    if args.node_means_only:
        print(json.dumps(node_means_leg(rr, synth, sync)))
        return
    if args.c2_only or args.c2_path_only:
        ctx = rr.Context(0)
        print(json.dumps(c2_legs(rr, synth, ctx, sync, steps=args.steps, path_only=args.c2_path_only)))
        ctx.close()
        return
    if args.generated_only:
        print(json.dumps(generated_scenarios_leg(rr, synth, sync, steps=args.steps)))
        return
    w = synth.config_c3()
    b, pf = w.basis, w.portfolio
    ctx = rr.Context(0)
    if args.term_bucket:
        ctx.set_option(rr.OPT_TERM_BUCKET, args.term_bucket)
    ctx.set_option(rr.OPT_LANE_SPREAD, args.lane_spread)
    ctx.set_option(rr.OPT_CURVE_SHARE, args.curve_share)
    t0 = time.perf_counter()
    ctx.basis_upload(b.q, b.v, b.shock)
    ctx.portfolio_upload(pf)
    sync()
    upload_s = time.perf_counter() - t0
    out = ctx.alloc_outputs(1, b.n_scen, stats=True)
    ctx.set_option(rr.OPT_BLOCK_K, args.block_k)
    ctx.set_option(rr.OPT_WG_PER_CU, args.wg)
    ctx.set_option(rr.OPT_BLOCK_J, args.block_j)
    ctx.set_option(rr.OPT_CURVE_RING, args.ring)

    def step():
        ctx.reserve_recurrence(0, 1, 0, b.n_scen, 12, out)

    t0 = time.perf_counter()
    step()                       # first call: launched directly (by the recurrence kernel: plan, autotune)
    sync()
    first_call_s = time.perf_counter() - t0
    for _ in range(args.warmup):
        step()
    sync()
    elapsed = timed_steps(step, args.steps, sync)
    ms_per_step = 1e3 * elapsed / args.steps
    # The paper's protocol (minimum of 7 runs): seven single steps, each
    # between HIP events on the stream the library launches on (the null
    # stream, torch's default stream here).
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(7)]
    for e0, e1 in evs:
        e0.record()
        step()
        e1.record()
    sync()
    step_ms7 = np.array([e0.elapsed_time(e1) for e0, e1 in evs])
    flops, ops, live, vsteps = scenario_step_work(pf)
    n_val = live * b.n_scen
    value = n_val / (elapsed / args.steps)
    if args.surrogate_only:
        ctx.close()
        ctx = rr.Context(0)
        r = surrogate_leg(rr, synth, ctx, w, None, n_val, ms_per_step, args.steps, sync,
                          profile_only=True, epochs=args.surrogate_epochs)
        print(json.dumps(r))
        ctx.close()
        return
    if args.kernel_only:
        print(json.dumps({"ms_per_step": ms_per_step, "value": value,
                          "block_k": ctx.get_option(rr.OPT_LAST_K),
                          "block_j": ctx.get_option(rr.OPT_LAST_J),
                          "wg_per_cu": ctx.get_option(rr.OPT_LAST_WG),
                          "curve_ring": ctx.get_option(rr.OPT_LAST_RING),
                          "windows": ctx.get_option(rr.OPT_LAST_WINDOWS)}))
        ctx.close()
        return

    # Second timed region: HIP events around every run's kernels (without the
    # totals pass and the statistic of the recurrence kernel's runs, and without
    # the statistic of runs by cash flows).
    ctx.set_option(rr.OPT_KERNEL_TIMING, 1)
    ctx.kernel_times()
    elapsed_direct = timed_steps(step, args.steps, sync)
    kms = ctx.kernel_times()
    ctx.set_option(rr.OPT_KERNEL_TIMING, 0)
    kernel_ms = float(np.mean(kms))
    k_opt = ctx.get_option(rr.OPT_LAST_K)
    by_flows = k_opt == 0      # no recurrence kernel: cash flows x discount products
    if by_flows:               # one multiply-add per valuation step, on the matrix cores
        flops, ops = 2 * vsteps, vsteps
    achieved = flops * b.n_scen / (kernel_ms * 1e-3) / 1e12
    issue_frac = None if by_flows else ops * b.n_scen / (kernel_ms * 1e-3) / FP64_ISSUE_PEAK
    wg_opt = ctx.get_option(rr.OPT_LAST_WG)
    j_opt = ctx.get_option(rr.OPT_LAST_J)
    ring_opt = ctx.get_option(rr.OPT_LAST_RING)
    traffic = measured_traffic(k_opt, j_opt, wg_opt, ring_opt)

    result = {
        "metric": "policy x scenario reserve valuations/s (exact FP64)",
        "value": value,
        "unit": "valuations/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic (seeded): GM mortality, Vasicek scenarios, mixed portfolio",
        "config": {"workload": w.name, "policies": pf.n, "scenarios": b.n_scen,
                   "max_steps": b.n_steps, "valuations_per_step": n_val,
                   "valuation_steps_per_step": vsteps * b.n_scen,
                   "outputs": "r0 [policy][scenario] + totals + tail statistic"},
        "roofline": {"bound": "mfma" if by_flows else "alu", "achieved": achieved, "peak": FP64_PEAK_TFLOPS,
                     "unit": "TFLOP/s", "frac": achieved / FP64_PEAK_TFLOPS, "traffic": traffic,
                     "kernel": "k_flow_sums, k_reserve_mm, k_flow_totals" if by_flows else "k_recurrence",
                     "kernel_ms": kernel_ms,
                     "kernel_launches": len(kms),
                     "algorithmic_flops_per_launch": flops * b.n_scen,
                     "algorithmic_bytes_per_launch": algorithmic_bytes(b, pf),
                     "issue_frac": issue_frac,
                     "flop_cap": flops / (2 * ops)},
        "valuation_steps_per_s": vsteps * b.n_scen / (elapsed / args.steps),
        "ms_per_step_direct_launch": 1e3 * elapsed_direct / args.steps,
        "step_ms_min_of_7": float(step_ms7.min()),
        "step_ms_median_of_7": float(np.median(step_ms7)),
        "first_call_s": first_call_s,
        "upload_s": upload_s,
        "launch": {"block_k": k_opt, "block_j": j_opt, "wg_per_cu": wg_opt,
                   "curve_ring": ctx.get_option(rr.OPT_LAST_RING),
                   "windows": ctx.get_option(rr.OPT_LAST_WINDOWS),
                   "by_cash_flows": by_flows, "autotuned": args.block_k == 0 and not by_flows},
    }

    exact_totals = out["totals"].cpu().numpy()[0]
    if not args.no_surrogate:
        ctx.close()
        ctx = rr.Context(0)
        result["surrogate"] = surrogate_leg(rr, synth, ctx, w, exact_totals, n_val, ms_per_step,
                                            args.steps, sync, epochs=args.surrogate_epochs)

    if not args.no_secondary:
        sec = {}
        ctx.close()
        ctx = rr.Context(0)
        sec.update(c2_legs(rr, synth, ctx, sync))
        ctx.close()
        ctx = rr.Context(0)
        w4 = synth.config_c4()
        ctx.basis_upload(w4.basis.q, w4.basis.v, w4.basis.shock)
        ctx.portfolio_upload(w4.portfolio)
        o4 = ctx.alloc_outputs(w4.basis.n_nodes, w4.basis.n_scen, r0=False, stats=True)
        f4 = lambda: ctx.reserve_recurrence(0, w4.basis.n_nodes, 0, w4.basis.n_scen, 12, o4)
        for _ in range(3):
            f4()
        e4 = timed_steps(f4, 10, sync)
        live4 = sum(int((w4.portfolio.term_m - 12 * k > 0).sum()) for k in range(w4.basis.n_nodes))
        ctx.set_option(rr.OPT_KERNEL_TIMING, 1)
        ctx.kernel_times()
        timed_steps(f4, 10, sync)
        k4 = float(np.mean(ctx.kernel_times()))
        ctx.set_option(rr.OPT_KERNEL_TIMING, 0)
        flops4 = sum(scenario_step_work(w4.portfolio, k, 12)[0] for k in range(w4.basis.n_nodes))
        flops4 *= w4.basis.n_scen
        chains4 = ctx.get_option(rr.OPT_LAST_K) > 0   # else summed cash flows: other work
        sec["C4_nested_60_nodes"] = {"valuations_per_s": live4 * w4.basis.n_scen / (e4 / 10) if chains4 else None,
                                     "node_scenario_totals_per_s":
                                     w4.basis.n_nodes * w4.basis.n_scen / (e4 / 10),
                                     "ms_per_step": 1e3 * e4 / 10,
                                     "live_valuations": live4 * w4.basis.n_scen,
                                     "nominal_valuations": w4.portfolio.n * w4.basis.n_nodes * w4.basis.n_scen,
                                     "kernel_ms": k4,
                                     "algorithmic_flops_per_launch": flops4,
                                     "kernel_tflops": flops4 / (k4 * 1e-3) / 1e12 if chains4 else None,
                                     "kernel_frac_fp64_peak": flops4 / (k4 * 1e-3) / 1e12 / FP64_PEAK_TFLOPS
                                     if chains4 else None,
                                     "launch": {"block_k": ctx.get_option(rr.OPT_LAST_K),
                                                "block_j": ctx.get_option(rr.OPT_LAST_J),
                                                "wg_per_cu": ctx.get_option(rr.OPT_LAST_WG)}}
        if not args.no_cpu:
            # The nested valuation on the host once, in full (reduced mode,
            # the process's CPU share): the CPU side of this secondary line.
            import oracle
            t0 = time.perf_counter()
            oracle.reserves_reduced(w4.basis, w4.portfolio, 0, w4.basis.n_nodes, 0, w4.basis.n_scen,
                                    12, n_threads=cpu_share(), want_r=False)
            c4s = time.perf_counter() - t0
            sec["C4_nested_60_nodes"]["cpu_reduced_mode"] = {
                "seconds": c4s, "valuations_per_s": live4 * w4.basis.n_scen / c4s,
                "threads": cpu_share(), "sample": "the whole workload, once"}
        sec["representative_500k_annuities"] = representative_leg(rr, synth, sync)
        sec["C3_device_generated_scenarios"] = generated_scenarios_leg(rr, synth, sync)
        sec["C4_node_means"] = node_means_leg(rr, synth, sync)
        result["secondary"] = sec
    ctx.close()

    if not args.no_cpu:
        result["cpu_baseline"] = cpu_baseline(w)
    print(json.dumps(result))


if __name__ == "__main__":
    main()
