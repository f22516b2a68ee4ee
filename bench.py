"""Benchmark: FoX attention forward + backward with ACP on one MI355X.

One step = fox_attn_fwd (boundary stage included, as the paper times it) +
fox_attn_bwd on the 760M-shaped layer (B=2, H=24, L=16384, d=64, bf16: the
16k-token end of the metric's 4k-16k range, and its largest savings), with all
inputs already in HBM.  Prints one JSON line.

    python bench.py [--gpus 1] [--steps 20] [--warmup 5] [--workload 760m]
                    [--no-cpu-baseline] [--no-decode] [--no-extra]

The line also carries the 125M/360M-shaped and adversarial layers, each with its
speedup over nothing pruned and the roofline of its dominant kernel (unless
--no-extra), decoding measurements (fox_attn_decode on the 125M layer shape) and
the Q/K projection (unless --no-decode), and the runtime reduction the paper
reports, as context.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "FoX attn fwd+bwd ms & effective TFLOP/s at L=4k-16k; % blocks pruned; MFMA util"
# What the paper reports for its own kernels (Sec. 4 and App. D), quoted as context only:
# other hardware, trained models and real gates instead of synthetic ones.
PAPER_CONTEXT = {
    "attention_runtime_reduction": "about 50-70% (2-3x) for one forward + backward, boundary search "
                                   "included",
    "boundary_search_share": "2-6% of the attention-kernel time (L = 4k-16k)",
    "setting": "Triton kernels on NVIDIA L40S (325 W), bf16, trained FoX (Pro) 125M/360M/760M at "
               "L = 4k/8k/16k",
}
PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
NOMINAL_CLOCK_GHZ = 2.4     # the shader clock the dense peak is quoted at
PEAK_HBM_GBS = 8000.0


def _flops(w, kept_tiles):
    dense_eff = 7.0 * w.B * w.H * w.L * w.L * w.d            # dense causal fwd + bwd
    per_tile = 64 * 64 * w.d
    return {
        "effective": dense_eff,
        "executed": kept_tiles * 14.0 * per_tile,             # fwd 4 + bwd 10 units per tile
        "fwd": kept_tiles * 4.0 * per_tile,
        "dkdv": kept_tiles * 8.0 * per_tile,                  # S, dP recompute + dV + dK
        "dq": kept_tiles * 2.0 * per_tile,                    # dQ (its S, dP recompute extra)
    }


def roofline(w, r):
    """The dominant attention kernel of a timed run and its rate: algorithmic
    FLOPs per launch (kept tiles x its units of 64 x 64 x d) over the mean
    launch duration from the library's own HIP events."""
    fl = _flops(w, r["kept"])
    pk = r["per_kernel_ms"]
    dom = max(("fwd", "dq", "dkdv"), key=lambda k: pk[k])
    achieved = fl[dom] / (pk[dom] * 1e-3) / 1e12
    out = {"bound": "mfma", "kernel": dom, "achieved": round(achieved, 2),
           "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
           "frac": round(achieved / PEAK_BF16_TFLOPS, 4),
           "traffic": measured_traffic(dom, w.name)}
    # The same rate against the shader clock the kernel sustains under this load
    # (from the counter profile; the nominal peak assumes 2.4 GHz), or None.
    clk = _profile_value("clock", dom, w.name)
    out["clock_ghz"] = clk
    out["frac_at_clock"] = (round(achieved / (PEAK_BF16_TFLOPS * clk / NOMINAL_CLOCK_GHZ), 4)
                            if clk else None)
    return out


def frac_at_step_clock(w, pk: dict, executed_tflops: float):
    """The step's executed MFMA rate against the peak at the clock its attention
    kernels sustain: their profiled clocks weighted by their share of the step's
    attention time; None unless all three have a current clock line."""
    ks = ("fwd", "dq", "dkdv")
    clocks = [_profile_value("clock", k, w.name) for k in ks]
    if any(c is None for c in clocks) or sum(pk[k] for k in ks) <= 0:
        return None
    clk = sum(pk[k] * c for k, c in zip(ks, clocks)) / sum(pk[k] for k in ks)
    return round(executed_tflops / (PEAK_BF16_TFLOPS * clk / NOMINAL_CLOCK_GHZ), 4)


# device headers that every kernel file includes: a change there changes the kernels
SHARED_HEADERS = ("acp_device.h", "acp_internal.h", "acp_rules.h", "acp_schedule.h")


def source_digest(src: str):
    """First 12 hex digits of the SHA-1 of a kernel source file followed by the
    shared device headers, or None when the file does not exist."""
    import hashlib
    d = os.path.join(ROOT, "paper_2504_06949_amd", "csrc")
    path = os.path.join(d, src)
    if not os.path.exists(path):
        return None
    h = hashlib.sha1(open(path, "rb").read())
    for name in SHARED_HEADERS:
        hp = os.path.join(d, name)
        if os.path.exists(hp):
            h.update(open(hp, "rb").read())
    return h.hexdigest()[:12]


def _profile_value(kind: str, kernel: str, workload: str):
    """A machine-read line `kind kernel workload value src:digest` of the committed
    rocprofv3 summaries, as a number, or None when none exists or the kernel's
    source changed since the counters were taken."""
    import glob
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", "*.md"))):
        for line in open(path):
            f = line.split()
            if len(f) == 5 and f[0] == kind and f[1] == kernel and f[2] == workload:
                src, digest = f[4].split(":")
                if source_digest(src) != digest:
                    return None
                return int(f[3]) if kind == "traffic" else float(f[3])
    return None


def measured_traffic(kernel: str, workload: str):
    """HBM bytes per launch of `kernel` on `workload` from the committed rocprofv3
    summaries (FETCH_SIZE + WRITE_SIZE, copy-calibrated), or None when none exists
    or the kernel's source changed since the counters were taken."""
    return _profile_value("traffic", kernel, workload)


def _stage1_ms(pk: dict) -> float:
    """Stage 1 per step: row norms (when they run), the plan and the workgroup
    schedule."""
    return pk["rownorm"] + pk["plan"] + pk.get("schedule", 0.0)


def _hbm_gbps(w, pk: dict) -> dict:
    """Achieved HBM rates of the memory-bound kernels from their compulsory bytes:
    row norms read Q and K; the plan reads log f and writes c (plus L/64-sized
    tables); the dlog f scan reads the row and column sums and writes dlog f."""
    bhl = w.B * w.H * w.L
    s = 2 if w.dtype == "bf16" else 4
    nbytes = {"rownorm": 2 * bhl * w.d * s, "plan": 8 * bhl, "dlogf": 12 * bhl}
    return {k: round(v / (pk[k] * 1e-3) / 1e9, 1) for k, v in nbytes.items() if pk.get(k)}


def run_workload(name, steps: int, warmup: int, eps_override=None, unpruned=True):
    """Time fwd+bwd steps of a named workload (or a Workload); QK-norm workloads
    take their bound from the norm scales (fox_attn_fwd_qknorm)."""
    import torch
    from paper_2504_06949_amd import acp, workloads

    w = workloads.WORKLOADS[name] if isinstance(name, str) else name
    x = workloads.generate(w)
    dev = torch.device("cuda:0")
    g = {k: (v.to(dev) if torch.is_tensor(v) else v) for k, v in x.items()}
    eps = w.eps if eps_override is None else eps_override
    ws = acp.workspace(g["q"])
    o = torch.empty_like(g["q"])
    lse = torch.empty(g["log_f"].shape, dtype=torch.float32, device=dev)
    grads = (torch.empty_like(g["q"]), torch.empty_like(g["k"]), torch.empty_like(g["v"]),
             torch.empty(g["log_f"].shape, dtype=torch.float32, device=dev))

    def step(e):
        if w.qk_norm:
            acp.forward_qknorm(g["q"], g["k"], g["v"], g["log_f"], g["gamma_q"], g["gamma_k"], e,
                               ws=ws, out=(o, lse))
        else:
            acp.forward(g["q"], g["k"], g["v"], g["log_f"], e, ws=ws, out=(o, lse))
        acp.backward(g["q"], g["k"], g["v"], o, g["do"], ws, out=grads)

    def timed(e):
        for _ in range(warmup):
            step(e)
        torch.cuda.synchronize()
        t0 = torch.cuda.Event(enable_timing=True)
        t1 = torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(steps):
            step(e)
        t1.record()
        torch.cuda.synchronize()
        return t0.elapsed_time(t1) / steps

    # one settling pass first: after the host-side set-up the clocks keep rising for
    # some milliseconds, which would make whichever timing came first read slow
    timed(eps)
    ms = timed(eps)
    # per-kernel durations from HIP events the library records on this stream,
    # over the same number of steps, right after the timed ones
    acp.acp_timing_enable(True)
    acp.acp_timing_reset()
    for _ in range(steps):
        step(eps)
    torch.cuda.synchronize()
    kt = acp.acp_timing_read()
    acp.acp_timing_enable(False)
    per_kernel = {k: (v[1] / v[0] if v[0] else 0.0) for k, v in kt.items()}
    # (read before the eps = 0 run replaces the plan in the workspace)
    kept = int(acp.plan_views(ws, w.B, w.H, w.L, w.d, g["q"].dtype)["kept"].sum().item())
    ms_dense = timed(0.0) if unpruned else float("nan")
    causal = w.B * w.H * w.M * (w.M + 1) // 2
    return {"w": w, "ms": ms, "ms_dense": ms_dense, "kept": kept, "causal": causal,
            "per_kernel_ms": per_kernel, "x": x}


def run_decode(steps: int = 64, warmup: int = 16, L0: int = 4096, C: int = 8192):
    """Decoding on the 125M-shaped layer (B=8, H=12, d=64, bf16, QK-normed q/k):
    a 4096-token prompt, then single-token steps with ACP (eps = e^-10, threshold
    sized for L_max = C) and with eps = 0.  After `warmup` eager steps, `steps`
    eager steps give the wall time per call (host side included), then `steps`
    more are captured in a HIP graph and replayed once: the replay time per step
    is the GPU time of the step's two kernels without the host's launch latency."""
    import torch
    from paper_2504_06949_amd import acp, workloads

    w0 = workloads.WORKLOADS["125m"]
    n_tok = warmup + 2 * steps
    L = L0 + 64 * ((n_tok + 63) // 64)
    dev = torch.device("cuda:0")
    if L0 <= 4096:
        w = workloads.custom("125m_decode", w0.B, w0.H, L, w0.d, "bf16", w0.seed, qk_norm=True)
        x = workloads.generate(w, with_grad=False)
        g = {n: x[n].to(dev) for n in ("q", "k", "v", "log_f", "gamma_q", "gamma_k")}
    else:
        # long prompts: drawn on the GPU (timing only)
        w = workloads.custom("125m_decode", w0.B, w0.H, L, w0.d, "bf16", w0.seed, qk_norm=True)
        g = workloads.long_decode_inputs(w0.B, w0.H, L, w0.d, w0.seed, dev)
    prompt = {n: g[n][:, :, :L0].contiguous() for n in ("k", "v", "log_f")}
    toks = [{n: g[n][:, :, t].contiguous() for n in ("q", "k", "v", "log_f")}
            for t in range(L0, L0 + n_tok)]
    out = {"workload": f"B={w.B} H={w.H} d={w.d} bf16, prompt {L0}, ring C={C}, L_max={C}, "
                       f"{steps} eager + {steps} graph-replayed steps after {warmup}"}
    o = torch.empty((w.B, w.H, w.d), dtype=torch.bfloat16, device=dev)
    lse = torch.empty((w.B, w.H), dtype=torch.float32, device=dev)
    row_bytes = 2 * w.d * 2 + 4                      # k and v rows plus c, per key
    for label, eps in (("acp", w.eps), ("unpruned", 0.0)):
        dec = acp.Decoder(w.B, w.H, C, w.d, dtype=torch.bfloat16, device=dev)
        dec.init(prompt["k"], prompt["v"], prompt["log_f"], g["gamma_q"], g["gamma_k"], eps, C)
        for tk in toks[:warmup]:
            dec.step(tk["q"], tk["k"], tk["v"], tk["log_f"], out=(o, lse))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for tk in toks[warmup:warmup + steps]:
            dec.step(tk["q"], tk["k"], tk["v"], tk["log_f"], out=(o, lse))
        torch.cuda.synchronize()
        wall = (time.perf_counter() - t0) / steps
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for tk in toks[warmup + steps:]:
                dec.step(tk["q"], tk["k"], tk["v"], tk["log_f"], out=(o, lse))
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        graph.replay()
        e1.record()
        torch.cuda.synchronize()
        gpu_us = e0.elapsed_time(e1) * 1e3 / steps
        t_last = dec.t - 1
        ptr = dec.current_pointer().long().cpu()
        lo = torch.clamp(64 * ptr, min=t_last - C + 1)
        keys = int((t_last - lo + 1).sum())
        nbytes = keys * row_bytes
        out[label] = {"step_us": round(gpu_us, 2), "wall_us_per_step": round(wall * 1e6, 1),
                      "keys_read": keys, "bytes_read": nbytes,
                      "hbm_gbps": round(nbytes / (gpu_us * 1e-6) / 1e9, 1),
                      "hbm_frac": round(nbytes / (gpu_us * 1e-6) / 1e9 / PEAK_HBM_GBS, 4),
                      "flags_or": int(dec.views()["flags"].max().item())}
        del graph, dec
    out["speedup_vs_unpruned"] = round(out["unpruned"]["step_us"] / out["acp"]["step_us"], 3)
    out["kv_reads_pruned_fraction"] = round(1 - out["acp"]["keys_read"] / out["unpruned"]["keys_read"], 4)
    return out


def run_projection(reps: int = 20, d_model: int = 768):
    """The Q/K projection with the norm epilogue on the 125M-shaped layer
    (X [B*L, d_model] bf16, Wq and Wk [d_model, H*d], d_model = 768 as in the
    paper's 125M model), against torch's bf16 matmul of the same product (no
    epilogue, row-major output) and the norm pass it makes unnecessary."""
    import torch
    from paper_2504_06949_amd import acp, workloads

    w0 = workloads.WORKLOADS["125m"]
    B, L, H, d = w0.B, w0.L, w0.H, w0.d
    p = workloads.projection_inputs(B, L, d_model, H, d, seed=7)
    dev = torch.device("cuda:0")
    x, wq, wk = (p[n].to(dev) for n in ("x", "wq", "wk"))
    q = torch.empty((B, H, L, d), dtype=torch.bfloat16, device=dev)
    k = torch.empty_like(q)
    ws = torch.empty(acp.acp_workspace_size(B, H, L, d, acp.ACP_BF16), dtype=torch.uint8,
                     device=dev)
    wqk = torch.cat([wq, wk], dim=1).contiguous()

    def timed(fn):
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / reps

    us = timed(lambda: acp.project_qk(x, wq, wk, B, H, d, ws=ws, out=(q, k)))
    mm_us = timed(lambda: torch.matmul(x, wqk))
    flops = 2.0 * 2 * (B * L) * d_model * (H * d)
    return {"workload": f"X [{B * L}, {d_model}] bf16 -> Q, K [{B}, {H}, {L}, {d}], "
                        f"norm maxima per 128-row chunk in the epilogue",
            "us": round(us, 2), "tflops": round(flops / (us * 1e-6) / 1e12, 1),
            "frac": round(flops / (us * 1e-6) / 1e12 / PEAK_BF16_TFLOPS, 4),
            "torch_matmul_us": round(mm_us, 2)}


def run_gate_fusion(reps: int = 20, d_model: int = 768):
    """The forget-gate producer with c in its epilogue on the 125M-shaped layer
    (X [B*L, d_model] bf16, d_model = 768 as in the paper's 125M model): its own
    time, the stage-1 plan kernel after it (no scan) against the plan kernel that
    scans log f, and the unfused sequence a model would otherwise run (torch's
    bf16 matmul for the gate logits, a log-sigmoid, and stage 1 with its scan)."""
    import torch
    from paper_2504_06949_amd import acp, workloads

    w = workloads.WORKLOADS["125m"]
    B, L, H, d = w.B, w.L, w.H, w.d
    p = workloads.gate_inputs(B, L, d_model, H, seed=9)
    dev = torch.device("cuda:0")
    x, wf, bf = (p[n].to(dev) for n in ("x", "w_f", "b_f"))
    g = {k: v.to(dev) for k, v in workloads.generate(w).items() if torch.is_tensor(v)}
    ws = acp.workspace(g["q"])
    lf = torch.empty((B, H, L), dtype=torch.float32, device=dev)
    o = torch.empty_like(g["q"])
    lse = torch.empty((B, H, L), dtype=torch.float32, device=dev)
    grads = (torch.empty_like(g["q"]), torch.empty_like(g["k"]), torch.empty_like(g["v"]),
             torch.empty((B, H, L), dtype=torch.float32, device=dev))

    def timed(fn, n=reps):
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / n

    def gated_step():
        acp.gate_project(x, wf, bf, B, H, d, ws=ws, log_f=lf)
        acp.forward_gated(g["q"], g["k"], g["v"], w.eps, ws, out=(o, lse))
        acp.backward(g["q"], g["k"], g["v"], o, g["do"], ws, out=grads)

    def plain_step():
        acp.forward(g["q"], g["k"], g["v"], lf, w.eps, ws=ws, out=(o, lse))
        acp.backward(g["q"], g["k"], g["v"], o, g["do"], ws, out=grads)

    gate_us = timed(lambda: acp.gate_project(x, wf, bf, B, H, d, ws=ws, log_f=lf))
    step_us = timed(gated_step)
    acp.acp_timing_enable(True)
    for label, fn in (("gated", gated_step), ("plain", plain_step)):
        acp.acp_timing_reset()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        kt = acp.acp_timing_read()
        pk = {k: (v[1] / v[0] * 1e3 if v[0] else 0.0) for k, v in kt.items()}
        if label == "gated":
            pk_g = pk
        else:
            pk_p = pk
    acp.acp_timing_enable(False)
    mm_us = timed(lambda: torch.nn.functional.logsigmoid(
        torch.matmul(x, wf).float() + bf).view(B, L, H).permute(0, 2, 1).contiguous())
    stage1_g = pk_g["rownorm"] + pk_g["plan"] + pk_g["schedule"]
    return {"workload": f"X [{B * L}, {d_model}] bf16, w_f [{d_model}, {H}] -> log f, c "
                        f"[{B}, {H}, {L}]; then fwd + bwd of the 125m layer",
            "gate_us": round(gate_us, 2),
            "plan_after_gate_us": round(pk_g["plan"], 2),
            "plan_with_scan_us": round(pk_p["plan"], 2),
            "fused_us": round(gate_us + pk_g["plan"], 2),
            "unfused_us": round(mm_us + pk_p["plan"], 2),
            "torch_gate_logits_us": round(mm_us, 2),
            "step_ms": round(step_us / 1e3, 4),
            "stage1_share": round(stage1_g * 1e-3 / (step_us / 1e3), 4),
            "gate_share": round(gate_us / step_us, 4)}


def cpu_baseline(res, budget_s: float = 15.0):
    """The oracle, untuned, on whole heads of the same workload until the budget is spent."""
    import numpy as np
    import oracle as orc
    from paper_2504_06949_amd import workloads

    try:
        from threadpoolctl import threadpool_info
        blas = [p.get("num_threads", 1) for p in threadpool_info() if p.get("user_api") == "blas"]
        cores = max(blas) if blas else 1
    except Exception:  # pragma: no cover
        cores = 1
    nproc = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    w, x = res["w"], res["x"]
    heads = [(b, h) for b in range(w.B) for h in range(w.H)]
    t0 = time.perf_counter()
    done = 0
    for b, h in heads:
        q, k, v, do = (workloads.to_f64(x[n][b, h]) for n in ("q", "k", "v", "do"))
        orc.run_head(q, k, v, x["log_f"][b, h].numpy(), w.eps, do=do)
        done += 1
        if time.perf_counter() - t0 >= budget_s:
            break
    dt = time.perf_counter() - t0
    per_head_eff = 7.0 * w.L * w.L * w.d
    return {"value": per_head_eff * done / dt / 1e12, "unit": "TFLOP/s (effective)",
            "cores": int(cores), "nproc": int(nproc),
            "omp_threads": os.environ.get("OMP_NUM_THREADS"), "kind": "oracle",
            "sample": f"{done} of {w.B * w.H} heads, full fwd+bwd per head in float64 "
                      f"({dt:.1f} s; extrapolates to {dt / done * w.B * w.H:.0f} s per step)"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="760m")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-decode", action="store_true",
                    help="skip the decoding measurement (125M-shaped, 4096-token prompt)")
    ap.add_argument("--skip-unpruned", action="store_true",
                    help="do not time the eps = 0 (nothing pruned) reference run")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="first run one plain device-to-device copy of MIB MiB (a known "
                         "byte count for calibrating HBM traffic counters under a profiler)")
    ap.add_argument("--no-extra", action="store_true",
                    help="skip the other layers (125M/360M/760M-shaped, adversarial)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: measures one GPU only (asked for --gpus {args.gpus}); "
              "the attention path shards over (batch, head) but no multi-GPU run is provided",
              file=sys.stderr)
        sys.exit(2)

    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)

    if args.copy_probe > 0:
        n = args.copy_probe * (1 << 20) // 4
        a = torch.ones(n, dtype=torch.float32, device="cuda:0")
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        del a, b
    res = run_workload(args.workload, args.steps, args.warmup, unpruned=not args.skip_unpruned)
    w = res["w"]
    fl = _flops(w, res["kept"])
    pk = res["per_kernel_ms"]
    names = {"125m": "125M", "360m": "360M", "760m": "760M"}
    out = {
        "metric": METRIC,
        "value": round(fl["effective"] / (res["ms"] * 1e-3) / 1e12, 2),
        "unit": "TFLOP/s (effective, dense-causal equivalent)",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(res["ms"], 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) Q/K/V/dO, gate logits N(mu_h, 0.5))",
        "config": {"workload": f"{names[w.name]}-shaped FoX layer: B={w.B} H={w.H} L={w.L} "
                               f"d={w.d}, eps=e^-10, 64x64 pruning grid" if w.name in names
                   else w.describe()},
        "pruned_fraction": round(1.0 - res["kept"] / res["causal"], 4),
        "executed_tflops": round(fl["executed"] / (res["ms"] * 1e-3) / 1e12, 2),
        "mfma_frac_executed": round(fl["executed"] / (res["ms"] * 1e-3) / 1e12
                                    / PEAK_BF16_TFLOPS, 4),
        "mfma_frac_executed_at_clock": frac_at_step_clock(
            w, pk, fl["executed"] / (res["ms"] * 1e-3) / 1e12),
        "ms_unpruned": None if args.skip_unpruned else round(res["ms_dense"], 4),
        "speedup_vs_unpruned": None if args.skip_unpruned else round(res["ms_dense"] / res["ms"], 3),
        "per_kernel_ms": {k: round(v, 4) for k, v in pk.items()},
        "boundary_share": round(_stage1_ms(pk) / res["ms"], 4),
        "hbm_gbps": _hbm_gbps(w, pk),
        "roofline": roofline(w, res),
    }
    if not args.no_extra:
        extra = {}
        for name in ("125m", "360m", "760m", "adv"):
            if name == w.name:
                continue
            r = run_workload(name, args.steps, args.warmup)
            f = _flops(r["w"], r["kept"])
            ex = f["executed"] / (r["ms"] * 1e-3) / 1e12
            extra[name] = {"ms": round(r["ms"], 3), "ms_unpruned": round(r["ms_dense"], 3),
                           "speedup_vs_unpruned": round(r["ms_dense"] / r["ms"], 3),
                           "effective_tflops": round(f["effective"] / (r["ms"] * 1e-3) / 1e12, 1),
                           "executed_tflops": round(ex, 1),
                           "mfma_frac_executed": round(ex / PEAK_BF16_TFLOPS, 4),
                           "mfma_frac_executed_at_clock": frac_at_step_clock(r["w"], r["per_kernel_ms"], ex),
                           "pruned_fraction": round(1 - r["kept"] / r["causal"], 4),
                           "boundary_share": round(_stage1_ms(r["per_kernel_ms"]) / r["ms"], 4),
                           "roofline": roofline(r["w"], r),
                           "per_kernel_ms": {k: round(v, 4) for k, v in r["per_kernel_ms"].items()}}
        # the 125m layer again with QK-normed queries and keys: the bound comes from
        # the norm scales and stage 1 makes no pass over Q and K
        from paper_2504_06949_amd import workloads as wl
        w125 = wl.WORKLOADS["125m"]
        wq = wl.custom("125m_qknorm", w125.B, w125.H, w125.L, w125.d, "bf16", w125.seed, qk_norm=True)
        r = run_workload(wq, args.steps, args.warmup)
        f = _flops(r["w"], r["kept"])
        rpk = r["per_kernel_ms"]
        extra["125m_qknorm"] = {"ms": round(r["ms"], 3), "ms_unpruned": round(r["ms_dense"], 3),
                                "speedup_vs_unpruned": round(r["ms_dense"] / r["ms"], 3),
                                "effective_tflops": round(f["effective"] / (r["ms"] * 1e-3) / 1e12, 1),
                                "pruned_fraction": round(1 - r["kept"] / r["causal"], 4),
                                "boundary_share": round(_stage1_ms(rpk) / r["ms"], 4),
                                "per_kernel_ms": {k: round(v, 4) for k, v in rpk.items()}}
        out["other_workloads"] = extra
    if not args.no_decode:
        out["decode"] = run_decode()
        # the regime App. F reports on: long prompts (the ring holds the whole
        # context, so every kept key is attended)
        out["decode_long"] = {str(n): run_decode(L0=n, C=n + 256) for n in (16384, 65536)}
        prj = run_projection()
        # the norm pass the fused epilogue replaces, as timed on the 125m layer
        pk125 = pk if w.name == "125m" else out.get("other_workloads", {}).get("125m", {}).get(
            "per_kernel_ms")
        prj["norm_pass_us_saved"] = round(pk125["rownorm"] * 1e3, 2) if pk125 else None
        out["projection"] = prj
        out["gate_fusion"] = run_gate_fusion()
    out["paper_context"] = PAPER_CONTEXT
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(res)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
