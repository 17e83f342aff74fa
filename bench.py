#!/usr/bin/env python3
"""Benchmark of the stick-breaking attention hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

A step is one pass of the hot path over one synthetic batch of the headline
workload (bf16, B=8, H=16, T=4096, d_head=128; half the heads with k*3): the
training forward (o and m) followed by the backward (dq, dk, dv).  Inputs are
resident in HBM before the timed region starts.  One JSON line is printed:
whole-step TFLOP/s as `value`, the forward and the two backward passes separately,
the same on inputs where no work can be left out, a roofline object for that
run's dominant kernel, every one of the five stated
workloads with its own timing and its error against the CPU oracle (`configs`),
the rate the matrix cores sustain on such data with no other work (the practical
ceiling under the power limit), the vendor GEMM at a large square shape and the
shader clock the forward ran at for context, and the CPU oracle timed on a
bounded sample.

FLOP convention (algorithmic, strictly causal pairs only): one contraction is
2*d FLOP per (query, key) pair with key < query; forward = 2 contractions,
backward = 5 (query-stationary pass: logits, dO.v, dQ = 3; key-stationary pass:
dK, dV = 2, its recomputation of the first two is not counted).  Nothing else
(masked halves of diagonal tiles, recomputation, element-wise work) is counted.
The kernels leave out terms whose weight is zero in fp32, and on the workload's
data (every stick is used up within tens of keys) those are most of them: `value`
and the rates of `fwd`, `bwd`, `configs` are EFFECTIVE rates, all pairs' operations
over the time, and may exceed what the hardware can execute.  `full_sweep` times the
same step on long-range inputs, where no term can be left out, and `roofline`
is of that run: these are achieved rates.

`roofline.traffic` (HBM bytes per launch of the dominant kernel) comes from
rocprofv3 counter runs that cannot be made from inside this script; it is read
from profiles/hbm_traffic_B8_H16_T4096_d128.txt (named in `traffic_source`) when
that file is present.  It is a stored measurement of the kernel as it was when the
profile was taken, not of this run; the file records fingerprints of the kernel sources it
was taken on, and `traffic_is_of_these_sources` says whether they are still the same.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0     # MI355X dense bf16 MFMA peak (published)
DEFAULT_PASSES = "fwd+bwd"


def flops_fwd(B, H, T, d):
    return 2.0 * B * H * d * T * (T - 1)


def flops_bwd(B, H, T, d):
    return 5.0 * B * H * d * T * (T - 1)


def event_time_ms(fn, iters):
    """Average duration of fn() over iters back-to-back launches, HIP events on
    the stream the kernels are launched on (torch's current stream)."""
    import torch
    for _ in range(2):                     # first use of a kernel pays for loading it
        fn()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(iters):
        fn()
    e1.record()
    e1.synchronize()
    return e0.elapsed_time(e1) / iters


def event_times_ms(fn, iters):
    """Per-launch durations: every launch bracketed by its own pair of events."""
    import torch
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(iters)]
    for a, b in ev:
        a.record()
        fn()
        b.record()
    ev[-1][1].synchronize()
    return sorted(a.elapsed_time(b) for a, b in ev)


def spread(ts):
    return {"ms_median": ts[len(ts) // 2], "ms_min": ts[0], "launches": len(ts)}


TRAFFIC_FILE = os.path.join("profiles", "hbm_traffic_B8_H16_T4096_d128.txt")
KERNEL_SOURCES = ("sb_fwd_bf16.hip", "sb_bwd_bf16.hip", "sb_decode.hip", "sb_split.h", "sb_mma.h", "sb_share.h")


def source_fingerprint(name):
    """sha256 of a kernel source with comments and white space removed: changes when the code does."""
    import hashlib
    import re
    with open(os.path.join(ROOT, "paper_2410_17980_amd", "csrc", name)) as f:
        text = f.read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    text = re.sub(r"//[^\n]*", "", text)
    return hashlib.sha256("".join(text.split()).encode()).hexdigest()[:16]


def _traffic_record():
    try:
        with open(os.path.join(ROOT, TRAFFIC_FILE)) as f:
            for line in f:
                if line.startswith("JSON:"):
                    return json.loads(line[5:])
    except OSError:
        pass
    return {}


def hbm_traffic(kernel):
    """HBM bytes per launch measured with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE (see the file)."""
    return _traffic_record().get(kernel)


def hbm_traffic_is_current():
    """True when the kernel sources are the ones the stored traffic figures were measured on."""
    want = _traffic_record().get("kernel_sources")
    if not want:
        return None
    try:
        return all(source_fingerprint(n) == h for n, h in want.items())
    except OSError:
        return None


def cpu_baseline(w, q, k, v, dout, n_heads, with_bwd):
    """The float64 oracle, as it stands, on n_heads (b, h) slices of the workload:
    forward and backward.  Reported in the metric's unit with the same FLOP formula."""
    from oracle import sb_oracle
    from paper_2410_17980_amd import inputs
    import torch
    sb_oracle.build()
    picks = inputs.slice_picks(w, n_heads)
    f64 = lambda t: t.to(torch.float32).to(torch.float64).numpy()
    qs, ks, vs, gs = ([f64(t[b, h]) for b, h in picks] for t in (q, k, v, dout))
    t0 = time.perf_counter()
    for i in range(n_heads):
        sb_oracle.fwd(qs[i], ks[i], vs[i])
    t1 = time.perf_counter()
    if with_bwd:
        for i in range(n_heads):
            sb_oracle.bwd(qs[i], ks[i], vs[i], gs[i])
    t2 = time.perf_counter()
    fl = n_heads * (flops_fwd(1, 1, w.T, w.d) + (flops_bwd(1, 1, w.T, w.d) if with_bwd else 0.0))
    return {
        "value": fl / (t2 - t0) / 1e12,
        "unit": "TFLOP/s",
        "cores": sb_oracle.num_threads(),
        "kind": "oracle",
        "sample": f"{n_heads} (b,h) slices of the workload, fwd {t1 - t0:.2f} s + bwd {t2 - t1:.2f} s, float64",
        "fwd_tflops": n_heads * flops_fwd(1, 1, w.T, w.d) / (t1 - t0) / 1e12,
        "bwd_tflops": n_heads * flops_bwd(1, 1, w.T, w.d) / (t2 - t1) / 1e12 if with_bwd else None,
        "extrapolated_full_workload_s": (t2 - t0) * w.B * w.H / n_heads,
    }


def launch_stats(fn, iters):
    """Mean over back-to-back launches plus median and minimum of individually timed ones."""
    ms = event_time_ms(fn, iters)
    return {"ms": ms, **spread(event_times_ms(fn, iters))}


def config_entries(sb, inputs, iters, headline):
    """The five stated workloads, each with its own launch timing (HIP events, >= 50
    launches) and its max abs error against the float64 oracle on the slices the
    workload states.  headline: (tensors, stats) of workload 3, measured by the caller."""
    import numpy as np
    import torch
    from oracle import sb_oracle
    sb_oracle.build()
    f64 = lambda t: t.detach().cpu().to(torch.float32).to(torch.float64).numpy()
    out = []
    for idx, w in enumerate(inputs.WORKLOADS):
        B, H, T, d = w.B, w.H, w.T, w.d
        e = {"config": idx + 1, "workload": w.name, "B": B, "H": H, "T": T, "d_head": d, "dtype": w.dtype,
             "pass": w.direction}
        if idx == 2:
            (q, k, v, _), st, od = headline
            qd = kd = vd = None
        else:
            ts = inputs.workload_tensors(w)
            q, k, v = ts[:3]
            qd, kd, vd = (t.cuda() for t in (q, k, v))
        if w.direction == "fwd":
            flop = flops_fwd(B, H, T, d)
            if w.dtype == "f32":
                od = torch.empty_like(qd)
                fn = lambda: sb.sb_attn_fwd_f32(qd, kd, vd, od)
                e["entry"], tol = "sb_attn_fwd_f32", 1e-5
            elif idx == 4:
                od = torch.empty_like(qd)
                fn = lambda: sb.sb_attn_fwd(qd, kd, vd, od)
                e["entry"], tol = "sb_attn_fwd", 2e-2
            elif idx != 2:
                od = torch.empty_like(qd)
                md = torch.empty((B, H, T), dtype=torch.float32, device="cuda")
                fn = lambda: sb.sb_attn_fwd_train(qd, kd, vd, od, md)
                e["entry"], tol = "sb_attn_fwd_train", 2e-2
            else:
                e["entry"], tol = "sb_attn_fwd_train", 2e-2
            if idx != 2:
                fn()
                st = launch_stats(fn, iters)
            # oracle check on the stated slices
            if idx == 0:
                ref, _ = sb_oracle.fwd(f64(q), f64(k), f64(v))
                err = float(np.abs(f64(od) - ref).max())
                e["checked"] = "all rows"
            elif idx == 4:
                picks, r0 = inputs.slice_picks(w, 2), T - 512
                err = 0.0
                for b, h in picks:
                    ref, _ = sb_oracle.fwd(f64(q[b, h]), f64(k[b, h]), f64(v[b, h]), rows=(r0, T))
                    err = max(err, float(np.abs(f64(od[b, h, r0:]) - ref).max()))
                e["checked"] = "2 heads, last 512 rows"
            else:
                picks = inputs.slice_picks(w, 4)
                err = 0.0
                for b, h in picks:
                    ref, _ = sb_oracle.fwd(f64(q[b, h]), f64(k[b, h]), f64(v[b, h]))
                    err = max(err, float(np.abs(f64(od[b, h]) - ref).max()))
                e["checked"] = "4 (b,h) slices" + (", 2 of them sharp heads" if w.sharp_half else "")
            e["max_abs_err"], e["tol"] = err, tol
        else:
            flop = flops_bwd(B, H, T, d)
            g = ts[3]
            gd = g.cuda()
            od, md = sb.sb_attn_fwd_train(qd, kd, vd)
            dq = torch.empty((B, H, T, d), dtype=torch.float32, device="cuda")
            dk, dv = torch.empty_like(dq), torch.empty_like(dq)
            ws = torch.empty(sb.sb_attn_bwd_workspace_bytes(B, H, T, d), dtype=torch.uint8, device="cuda")
            fn = lambda: sb.sb_attn_bwd(qd, kd, vd, md, gd, dq, dk, dv, ws)
            fn()
            st = launch_stats(fn, iters)
            e["entry"] = "sb_attn_bwd"
            picks = inputs.slice_picks(w, 4)
            errs = {"dq": 0.0, "dk": 0.0, "dv": 0.0}
            rels = {"dq": 0.0, "dk": 0.0, "dv": 0.0}
            for b, h in picks:
                refs = sb_oracle.bwd(f64(q[b, h]), f64(k[b, h]), f64(v[b, h]), f64(g[b, h]))
                for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
                    err1 = float(np.abs(f64(got[b, h]) - ref).max())
                    errs[name] = max(errs[name], err1)
                    rels[name] = max(rels[name], err1 / float(np.abs(ref).max()))
            e["checked"] = "4 (b,h) slices, analytic gradients"
            e["max_abs_err"], e["tol"] = max(errs.values()), 2e-2
            e["max_abs_err_by_tensor"], e["max_err_over_max_ref"] = errs, rels
        tf = flop / (st["ms"] * 1e-3) / 1e12
        e.update({"flop": flop, **st, "effective_tflops": tf, "effective_frac_bf16_peak": tf / PEAK_BF16_TFLOPS,
                  "ok": bool(e["max_abs_err"] <= e["tol"])})
        if w.dtype == "f32":
            e["note"] = "full-precision check path, latency-bound at this size: not a matrix-core rate"
        out.append(e)
    return out


def long_range(inputs, w):
    """q, k, v, dout of a workload's shape with logits about N(-6,1): the stick lasts for hundreds to
    thousands of keys and no term of the sweep is zero."""
    return [t.cuda() for t in inputs.biased_gaussian(w.B, w.H, w.T, w.d, seed=w.seed, shift=-6.0, with_dout=True)]


def run_one_config(sb, inputs, n, iters, calibrate_copy=False, far=False, with_bwd=False):
    """One stated workload on its own (training forward, plus the backward for the backward
    workload or on request), launched `iters` times: the command a rocprofv3 run of that shape wraps."""
    import torch
    w = inputs.WORKLOADS[n - 1]
    B, H, T, d = w.B, w.H, w.T, w.d
    if far:
        ts = long_range(inputs, w)
    elif with_bwd and w.direction == "fwd":
        ts = [t.cuda() for t in inputs.gaussian(B, H, T, d, w.seed, w.dtype, w.sharp_half, with_dout=True)]
    else:
        ts = [t.cuda() for t in inputs.workload_tensors(w)]
    q, k, v = ts[:3]
    if calibrate_copy:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.bitwise_or(src, 0, out=dst)
        torch.cuda.synchronize()
        del src, dst
    o = torch.empty_like(q)
    if w.dtype == "f32":
        fn = lambda: sb.sb_attn_fwd_f32(q, k, v, o)
    else:
        m = torch.empty((B, H, T), dtype=torch.float32, device="cuda")
        if w.direction == "fwd" and not with_bwd:
            fn = lambda: sb.sb_attn_fwd_train(q, k, v, o, m)
        else:
            dq = torch.empty((B, H, T, d), dtype=torch.float32, device="cuda")
            dk, dv = torch.empty_like(dq), torch.empty_like(dq)
            ws = torch.empty(sb.sb_attn_bwd_workspace_bytes(B, H, T, d), dtype=torch.uint8, device="cuda")

            def fn():
                sb.sb_attn_fwd_train(q, k, v, o, m)
                sb.sb_attn_bwd(q, k, v, m, ts[3], dq, dk, dv, ws)
    ms = event_time_ms(fn, iters)
    return {"config": n, "workload": w.name, "launches": iters, "ms": ms}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--cpu-heads", type=int, default=48, help="(b,h) slices the CPU oracle is timed on; 0 = skip")
    ap.add_argument("--kernel-iters", type=int, default=50, help="launches per kernel for the event timing")
    ap.add_argument("--passes", choices=["fwd", "fwd+bwd"], default=DEFAULT_PASSES,
                    help="what one step runs")
    ap.add_argument("--no-configs", action="store_true", help="skip the per-workload `configs` array")
    ap.add_argument("--only-config", type=int, default=0, metavar="N",
                    help="profiling aid: run only stated workload N (1-5) --kernel-iters times, print its timing "
                         "and exit (what a rocprofv3 run of one of the other shapes wraps)")
    ap.add_argument("--long-range", action="store_true", help="with --only-config: long-range inputs of that shape")
    ap.add_argument("--with-bwd", action="store_true", help="with --only-config: forward and backward")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run a plain 1 GiB element-wise copy kernel (3 times): the known traffic the "
                         "FETCH_SIZE / WRITE_SIZE counters of a rocprofv3 --pmc run are scaled by")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on one GPU; --gpus must be 1 (batch and heads shard "
                 "without communication, so N GPUs would each run this same kernel on B/N).")

    import torch
    from paper_2410_17980_amd import binding as sb
    from paper_2410_17980_amd import inputs

    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible")
    sb.load(build_if_missing=True)
    torch.cuda.set_device(0)

    if args.only_config:
        print(json.dumps(run_one_config(sb, inputs, args.only_config, args.kernel_iters, args.calibrate_copy,
                                        args.long_range, args.with_bwd)))
        return

    w = inputs.WORKLOADS[2]
    B, H, T, d = w.B, w.H, w.T, w.d
    q, k, v, dout = inputs.gaussian(B, H, T, d, w.seed, w.dtype, w.sharp_half, with_dout=True)
    qd, kd, vd, gd = (t.cuda() for t in (q, k, v, dout))
    o = torch.empty_like(qd)
    m = torch.empty((B, H, T), dtype=torch.float32, device="cuda")
    dq = torch.empty((B, H, T, d), dtype=torch.float32, device="cuda")
    dk = torch.empty_like(dq)
    dv = torch.empty_like(dq)
    ws = torch.empty(sb.sb_attn_bwd_workspace_bytes(B, H, T, d), dtype=torch.uint8, device="cuda")

    def fwd():
        sb.sb_attn_fwd_train(qd, kd, vd, o, m)

    def bwd():
        sb.sb_attn_bwd(qd, kd, vd, m, gd, dq, dk, dv, ws)

    with_bwd = args.passes == "fwd+bwd"

    if args.calibrate_copy:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.bitwise_or(src, 0, out=dst)      # a kernel (a plain copy_ may go through the DMA engines)
        torch.cuda.synchronize()
        del src, dst

    def step():
        fwd()
        if with_bwd:
            bwd()

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps

    f_fwd, f_bwd = flops_fwd(B, H, T, d), flops_bwd(B, H, T, d)
    ms_fwd = event_time_ms(fwd, args.kernel_iters)
    sp_fwd = spread(event_times_ms(fwd, args.kernel_iters))
    tf_fwd = f_fwd / (ms_fwd * 1e-3) / 1e12
    o_fwd = o.clone()                      # the headline forward's output, checked against the oracle below
    kernels = {"fwd_bf16_kernel": (ms_fwd, f_fwd)}
    if with_bwd:
        ms_bwd = event_time_ms(bwd, args.kernel_iters)
        sp_bwd = spread(event_times_ms(bwd, args.kernel_iters))
        ms_dq = event_time_ms(lambda: sb.sb_attn_bwd_dq(qd, kd, vd, m, gd, dq, ws), args.kernel_iters)
        ms_dkdv = event_time_ms(lambda: sb.sb_attn_bwd_dkdv(qd, kd, vd, gd, ws, dk, dv), args.kernel_iters)
        tf_bwd = f_bwd / (ms_bwd * 1e-3) / 1e12
        kernels["bwd_dq_kernel"] = (ms_dq, 0.6 * f_bwd)
        kernels["bwd_dkv_pair_kernel" if d == 128 else "bwd_dkv_kernel"] = (ms_dkdv, 0.4 * f_bwd)
    value = (f_fwd + (f_bwd if with_bwd else 0.0)) / (ms_per_step * 1e-3) / 1e12

    # early halt (inference forward; NOT part of the step or of `value`): how much of the sweep
    # the workload's data lets a block skip at eps = 1e-9, and what that buys
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    sb.sb_attn_fwd_halt(qd, kd, vd, 1e-9, o, counts)
    swept, full = counts.cpu().tolist()
    ms_inf = event_time_ms(lambda: sb.sb_attn_fwd(qd, kd, vd, o), args.kernel_iters)
    ms_halt = event_time_ms(lambda: sb.sb_attn_fwd_halt(qd, kd, vd, 1e-9, o), args.kernel_iters)

    # the same, and the step's kernels, on long-range inputs: no term can be left out
    ql, kl, vl, gl = long_range(inputs, w)
    full_kernels = {"fwd_bf16_kernel": (event_time_ms(lambda: sb.sb_attn_fwd_train(ql, kl, vl, o, m), args.kernel_iters), f_fwd)}
    if with_bwd:
        full_kernels["bwd_dq_kernel"] = (
            event_time_ms(lambda: sb.sb_attn_bwd_dq(ql, kl, vl, m, gl, dq, ws), args.kernel_iters), 0.6 * f_bwd)
        full_kernels["bwd_dkv_pair_kernel" if d == 128 else "bwd_dkv_kernel"] = (
            event_time_ms(lambda: sb.sb_attn_bwd_dkdv(ql, kl, vl, gl, ws, dk, dv), args.kernel_iters), 0.4 * f_bwd)
    counts.zero_()
    sb.sb_attn_fwd_halt(ql, kl, vl, 1e-9, o, counts)
    swept_l, full_l = counts.cpu().tolist()
    ms_inf_l = event_time_ms(lambda: sb.sb_attn_fwd(ql, kl, vl, o), args.kernel_iters)
    ms_halt_l = event_time_ms(lambda: sb.sb_attn_fwd_halt(ql, kl, vl, 1e-9, o), args.kernel_iters)
    # the other way to take Algorithm 1's in-tile cumulative sum: triangular-matrix MFMA in the
    # log domain (measurement variant, same outputs to the same tolerance)
    ms_tri = event_time_ms(lambda: sb.sb_diag_fwd_tri(ql, kl, vl, o, m), args.kernel_iters)
    ms_fwd_again = event_time_ms(lambda: sb.sb_attn_fwd_train(ql, kl, vl, o, m), args.kernel_iters)
    del ql, kl, vl, gl
    fwd()                                  # o and m of the workload again

    # single-token decode (NOT part of the step or of `value`): one query per head against a
    # cache of 16384 tokens; bound by HBM bandwidth, K and V are read once
    Td = 16384
    gd_ = torch.Generator(device="cpu")
    gd_.manual_seed(w.seed)
    kc = torch.randn(B, H, Td, d, generator=gd_, dtype=torch.float32).to(torch.bfloat16).cuda()
    vc = torch.randn(B, H, Td, d, generator=gd_, dtype=torch.float32).to(torch.bfloat16).cuda()
    q1 = qd[:, :, 0].contiguous()
    o1 = torch.empty_like(q1)
    wsd = torch.empty(sb.load().sb_attn_decode_workspace_bytes(B, H, Td, d), dtype=torch.uint8, device="cuda")
    ms_dec = event_time_ms(lambda: sb.sb_attn_decode(q1, kc, vc, o=o1, workspace=wsd), 3 * args.kernel_iters)
    # with m wanted every key is read, whatever the nearest ones take
    m1 = torch.empty((B, H), dtype=torch.float32, device="cuda")
    ms_dec_all = event_time_ms(lambda: sb.sb_attn_decode(q1, kc, vc, o=o1, m=m1, workspace=wsd), 3 * args.kernel_iters)
    dec_bytes = 2.0 * B * H * Td * d * 2
    # what a kernel that only reads the same number of bytes reaches (K and V together)
    kv_all = torch.cat([kc.reshape(-1), vc.reshape(-1)])
    stream_gbs = sb.sb_diag_stream_read(kv_all, iters=20)
    del kc, vc, kv_all

    # the rate the matrix cores sustain on data like the workload's with nothing else running
    mfma_tf, mfma_mhz = sb.sb_diag_mfma_rate(kd.reshape(-1)[: 1 << 21], iters=4000)

    # the shader clock the chip holds while the forward runs (sampled inside the kernel, after
    # a burst of launches so that the power management has settled)
    for _ in range(20):
        fwd()
    fwd_mhz = sb.sb_diag_fwd_clock(qd, kd, vd, o, m)

    # context: the vendor GEMM (hipBLASLt through torch.mm) on a large square bf16 problem
    n_g = 8192
    ga = torch.randn(n_g, n_g, device="cuda", dtype=torch.bfloat16)
    gb = torch.randn(n_g, n_g, device="cuda", dtype=torch.bfloat16)
    gc = torch.empty_like(ga)
    torch.mm(ga, gb, out=gc)
    ms_gemm = event_time_ms(lambda: torch.mm(ga, gb, out=gc), 20)
    gemm_tf = 2.0 * n_g ** 3 / (ms_gemm * 1e-3) / 1e12
    del ga, gb, gc

    # dominant kernel = the one with the largest share of the full sweep's step
    dom = max(full_kernels, key=lambda n: full_kernels[n][0])
    dom_ms, dom_flop = full_kernels[dom]
    dom_tf = dom_flop / (dom_ms * 1e-3) / 1e12

    out = {
        "metric": "stick-breaking attn fwd/bwd TFLOP/s + % bf16 MFMA peak, B8 H16 T4096 d128",
        "value": value,
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": "train_step_bf16_B8_H16_T4096_d128", "B": B, "H": H, "T": T, "d_head": d,
                   "inputs": "iid N(0,1) bf16, heads h>=H/2 with k*3, seed 2",
                   "step": "fwd_train + bwd" if with_bwd else "fwd_train",
                   "zero_weights": "terms whose weight is zero in fp32 are left out (exact); no halting threshold"},
        "rates": "value, fwd, bwd and configs: effective (all causal pairs' operations / time); full_sweep and "
                 "roofline: achieved (inputs on which no term is left out)",
        "fwd": {"ms": ms_fwd, "effective_tflops": tf_fwd, "effective_frac_bf16_peak": tf_fwd / PEAK_BF16_TFLOPS, **sp_fwd},
        "bwd": {"ms": ms_bwd, "effective_tflops": tf_bwd, "effective_frac_bf16_peak": tf_bwd / PEAK_BF16_TFLOPS,
                "dq_pass_ms": ms_dq, "dkdv_pass_ms": ms_dkdv, **sp_bwd} if with_bwd else None,
        "roofline": {"bound": "mfma", "kernel": dom, "achieved": dom_tf, "peak": PEAK_BF16_TFLOPS,
                     "unit": "TFLOP/s", "frac": dom_tf / PEAK_BF16_TFLOPS, "avg_launch_ms": dom_ms,
                     "flop_per_launch": dom_flop, "inputs": "long range: every term of the sweep counts",
                     "avg_launch_ms_on_workload": kernels[dom][0], "traffic": hbm_traffic(dom + "/full_sweep"),
                     "traffic_on_workload": hbm_traffic(dom)},
        "full_sweep": {"inputs": "N(0,1) q, k, v with a bias coordinate: logits about N(-6,1)",
                       "ms": sum(t for t, _ in full_kernels.values()),
                       "tflops": sum(f for _, f in full_kernels.values()) / sum(t for t, _ in full_kernels.values()) / 1e9,
                       "kernels": {n: {"ms": t, "tflops": f / t / 1e9, "frac_bf16_peak": f / t / 1e9 / PEAK_BF16_TFLOPS,
                                       "frac_mfma_only_ceiling": f / t / 1e9 / mfma_tf}
                                   for n, (t, f) in full_kernels.items()}},
        "early_halt": {"eps": 1e-9, "ms_no_threshold": ms_inf, "ms_halted": ms_halt, "speedup": ms_inf / ms_halt,
                       "tiles_swept_frac": swept / max(full, 1),
                       "note": "sb_attn_fwd_halt vs sb_attn_fwd (forward without m, which stops where every farther "
                               "weight is zero); depends on the data: N(0,1) logits exhaust the stick within a "
                               "few dozen keys"},
        "early_halt_long_range": {"eps": 1e-9, "ms_no_threshold": ms_inf_l, "ms_halted": ms_halt_l,
                                  "speedup": ms_inf_l / ms_halt_l, "tiles_swept_frac": swept_l / max(full_l, 1),
                                  "inputs": "N(0,1) q, k, v with a bias coordinate: logits about N(-6,1)"},
        "decode": {"workload": f"B{B} H{H} cache T{Td} d{d}, bf16, one query per head", "ms": ms_dec,
                   "effective_gbs": dec_bytes / (ms_dec * 1e-3) / 1e9, "ms_all_keys_read": ms_dec_all,
                   "note": "far keys of exhausted heads are not read; with m wanted (ms_all_keys_read) all are",
                   "roofline": {"bound": "hbm", "achieved": dec_bytes / (ms_dec_all * 1e-3) / 1e9, "peak": 8000.0,
                                "unit": "GB/s", "frac": dec_bytes / (ms_dec_all * 1e-3) / 1e9 / 8000.0,
                                "bytes_per_launch": dec_bytes, "what": "K and V read once, m wanted",
                                "traffic": hbm_traffic("decode_kernel/all_keys"),
                                "streaming_read_gbs": stream_gbs,
                                "frac_streaming_read": dec_bytes / (ms_dec_all * 1e-3) / 1e9 / stream_gbs}},
        "fwd_shader_clock_mhz": fwd_mhz,
        "cumsum_variants": {"in_lane_chain_ms": ms_fwd_again, "triangular_mfma_ms": ms_tri,
                            "what": "training forward at the headline shape on long-range inputs with the in-tile "
                                    "reverse cumulative sum as the in-lane linear-domain chain (product path) and "
                                    "as a triangular-ones MFMA in the log domain (sb_diag_fwd_tri), "
                                    "timed back to back"},
        "gemm_reference": {"tflops": gemm_tf, "frac_bf16_peak": gemm_tf / PEAK_BF16_TFLOPS, "ms": ms_gemm,
                           "what": "torch.mm (hipBLASLt), bf16, 8192^3, N(0,1) data: the vendor's dense "
                                   "contraction on this chip, for context"},
        "mfma_only_ceiling": {"tflops": mfma_tf, "frac_bf16_peak": mfma_tf / PEAK_BF16_TFLOPS,
                              "shader_clock_mhz": mfma_mhz,
                              "what": "32x32x16 bf16 MFMAs alone, operands = the workload's k, 2 waves per SIMD"},
    }
    # the achieved rate against what the matrix cores sustain on such data (measured above)
    out["roofline"]["frac_mfma_only_ceiling"] = dom_tf / mfma_tf
    out["roofline"]["traffic_source"] = TRAFFIC_FILE + " (stored rocprofv3 run)"
    # false: the kernel sources changed since that run, the figure describes an older kernel
    out["roofline"]["traffic_is_of_these_sources"] = hbm_traffic_is_current()
    out["full_sweep"]["kernels"]["fwd_bf16_kernel"]["frac_gemm_reference"] = f_fwd / full_kernels["fwd_bf16_kernel"][0] / 1e9 / gemm_tf
    if not args.no_configs:
        out["configs"] = config_entries(sb, inputs, max(args.kernel_iters, 50),
                                        ((q, k, v, dout), {"ms": ms_fwd, **sp_fwd}, o_fwd))
    if args.cpu_heads > 0:
        out["cpu_baseline"] = cpu_baseline(w, q, k, v, dout, args.cpu_heads, with_bwd)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
