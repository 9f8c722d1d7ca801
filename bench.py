#!/usr/bin/env python3
"""Throughput of the region-sparse DiT denoising step on one MI355X.

Workload (the largest single-GPU configuration): video DiT, 21 latent frames x
30 x 52 patches = 32760 tokens, 64 channels, hidden 1536, 12 heads x 128, MLP
6144, 30 blocks, bf16 weights; 140 regions of 3x6x13 tokens, 42 of them active
per step in a band that moves with the frame and the step (9828 active tokens).
Inputs (weights, K/V caches, latents, thresholds) are seeded synthetic data
resident in HBM before timing.  One step = region score, gate select, gather,
embed, 30 DiT blocks on the active rows, final layer, scatter-update, all
through the C ABI.  The image workload (4096 tokens, 24 blocks, 1664 active
rows) is timed the same way as a secondary figure.

Prints one JSON line: active tokens/s, ms/step, the roofline of the dominant
kernel (timed live with HIP events around its launches) and the CPU oracle's
throughput on a bounded sample of the same workload.
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

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0          # MI355X HBM3E
WORKLOAD = "video"


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--pool", type=int, default=4, help="distinct latent pairs cycled through")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--workload", default=WORKLOAD, help="video (default), image, audio, packed or tiny")
    ap.add_argument("--cpu-seconds", type=float, default=12.0, help="budget of the CPU oracle sample")
    ap.add_argument("--cpu-threads", type=int, default=None,
                    help="cap on the oracle's BLAS threads (default: every host core)")
    ap.add_argument("--no-hbm", action="store_true", help="skip the streaming-kernel bandwidth figures")
    ap.add_argument("--no-secondary", action="store_true", help="skip the secondary image-workload figure")
    ap.add_argument("--no-trajectory", action="store_true", help="skip the chained-trajectory study")
    ap.add_argument("--trajectory", type=int, default=0, metavar="T",
                    help="instead of the benchmark: T chained steps per threshold and skip mode, deviation "
                         "of the final latent from the dense trajectory (prints its own JSON line)")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="launch a plain fp32 copy of this many MiB 3 times first (counter calibration)")
    return ap.parse_args()


def kernel_flops(name: str, w, M: int) -> float:
    """Algorithmic flops of one launch of an MFMA kernel at M active rows."""
    D, F, C = w.D, w.F, w.C
    Nb = w.N // w.B
    return {"gemm_qkv": 2.0 * M * D * 3 * D, "gemm_o": 2.0 * M * D * D, "gemm_mlp1": 2.0 * M * D * F,
            "gemm_mlp2": 2.0 * M * F * D, "attn": 4.0 * M * Nb * D, "embed": 2.0 * M * C * D,
            "final": 2.0 * M * D * C}.get(name, 0.0)


def importance_cost(fdl, stp, run, w, M: int, i: int) -> dict:
    """Untimed: one step with the paper's importance signal computed from the last
    block's self-attention, the importance call bracketed by the library's event
    timer.  Flops: the |A_r|^2 in-region scores of every active region and head."""
    torch = sys.modules["torch"]
    orig = stp.step

    def step_imp(*a, **k):
        k["importance_block"] = w.L - 1
        return orig(*a, **k)

    stp.step = step_imp
    fdl.fd_timer_arm("importance", 8)
    run(i)
    torch.cuda.synchronize()
    ms = fdl.fd_timer_read(8)
    fdl.fd_timer_disarm()
    stp.step = orig
    n_act = int(stp.active.sum().item())
    region_tokens = M / max(n_act, 1)
    flops = n_act * region_tokens * region_tokens * w.H * 2.0 * w.dh
    us = float(ms.sum()) * 1e3
    return {"when": "once per step with the importance gate signal (not in the timed step)",
            "block": w.L - 1, "active_regions": n_act, "us": us, "flops": flops,
            "achieved_tflops": flops / (us * 1e-6) / 1e12 if us > 0 else None}


def partition_cost(torch, fdl, wl) -> dict:
    """Untimed: the patch partitioner, which runs once per request after the
    warm-up steps, on the workloads' synthetic saliency maps (every request of
    the batch in one call), each call bracketed by the library's event timer."""
    out = {"when": "once per request after the warm-up steps (not in the timed step)"}
    for name in ("image", "audio", "video", "packed"):
        w = wl.WORKLOADS[name]
        rm = wl.region_map(w)
        reg_off = np.concatenate([[0], np.cumsum([rq.n_regions for rq in w.requests])]).astype(np.int32)
        sal = torch.from_numpy(wl.saliency_maps(w).view(np.int16)).cuda()
        region = torch.empty(w.N, dtype=torch.int32, device="cuda")
        ws = torch.empty(max(fdl.fd_partition_ws_size(w.N, w.B), 256), dtype=torch.uint8, device="cuda")
        for _ in range(3):
            fdl.fd_partition(rm.req_tok_off, reg_off, sal, region, ws)
        torch.cuda.synchronize()
        fdl.fd_timer_arm("partition", 16)
        for _ in range(10):
            fdl.fd_partition(rm.req_tok_off, reg_off, sal, region, ws)
        torch.cuda.synchronize()
        ms = fdl.fd_timer_read(16)
        fdl.fd_timer_disarm()
        out[name] = {"requests": w.B, "tokens": w.N, "regions": int(reg_off[-1]),
                     "us": round(float(np.mean(ms)) * 1e3, 2)}
    return out


def kernel_bytes(name: str, w, M: int) -> float:
    """Algorithmic HBM bytes of one launch of a streaming kernel."""
    C, N = w.C, w.N
    return {"score": 2.0 * N * C * 4 + 8 * w.R, "gather": M * (C * 4 + C * 2 + 4),
            "scatter": M * (4 * C * 4 + 4)}.get(name, 0.0)


def hbm_streams(torch, fdl, wl, pool_bytes: float = 1.1 * 2**30) -> dict:
    """GB/s of the three streaming kernels (region score, gather, scatter-update)
    against the 8 TB/s HBM peak, each launch on its own buffers from a pool of more
    than 1 GiB cycled in order, so the 256 MB MALL cannot serve a launch from the
    previous ones.  Durations come from the library's event timer around each
    launch; bytes are the algorithmic ones.  Two figures: the image workload's own
    shape (one request, ~1-2 MB per launch, bound by launch and ramp latency) and one
    launch over 64 and over 256 such requests (the packed path scaled up, 40-540 MB
    per launch)."""
    shapes = {
        "image_1_request": wl.WORKLOADS["image"],
    }
    for nreq in (64, 256):
        shapes[f"image_{nreq}_requests"] = wl.Workload(
            f"image{nreq}", C=64, D=1536, H=24, dh=64, F=6144, L=24,
            requests=tuple(wl.RequestShape("grid2d", (64, 64), (8, 8)) for _ in range(nreq)),
            activity="count", activity_args=(26,), dt=-0.02, steps=50, seed=1239)
    out = {}
    for label, w in shapes.items():
        rm = wl.region_map(w)
        plan = fdl.make_plan(rm.token_region, rm.req_tok_off, rm.n_regions)
        inp = wl.step_inputs(w, 0, rmap=rm)
        act = inp.hot
        tok = np.nonzero(act[rm.token_region])[0].astype(np.int32)
        M = len(tok)
        idx = torch.zeros(w.N, dtype=torch.int32, device="cuda")
        idx[:M] = torch.from_numpy(tok).cuda()
        m = torch.tensor([M], dtype=torch.int32, device="cuda")
        active = torch.from_numpy(act.astype(np.uint8)).cuda()
        dt = torch.from_numpy(wl.dt_per_request(w)).cuda()
        lat_bytes = w.N * w.C * 4
        P = max(4, int(np.ceil(pool_bytes / (2 * lat_bytes))))
        xs = [torch.randn(w.N, w.C, device="cuda") for _ in range(2 * P)]       # P (x_cur, x_prev) pairs
        vs = [torch.randn(w.N, w.C, device="cuda") for _ in range(P)]           # velocities (first M rows)
        vcs = [torch.empty(w.N, w.C, device="cuda") for _ in range(P)]          # vcache
        xa = [torch.empty(w.N, w.C, dtype=torch.int16, device="cuda") for _ in range(P)]
        score = torch.empty(w.R, dtype=torch.float64, device="cuda")
        ws = torch.empty(fdl.fd_region_score_ws_size(plan, w.C), dtype=torch.uint8, device="cuda")
        launches = {
            "score": lambda i: fdl.fd_region_score(plan, w.C, xs[2 * i], xs[2 * i + 1], score, ws),
            "gather": lambda i: fdl.fd_gather(plan, w.C, xs[2 * i], idx, m, xa[i]),
            "scatter": lambda i: fdl.fd_scatter_update(plan, w.C, xs[2 * i + 1], vs[i], idx, m, dt, vcs[i], active,
                                                       fdl.FD_SKIP_FREEZE),
        }
        res = {"tokens": w.N, "requests": w.B, "active_tokens": M, "pool_bytes": 2 * P * lat_bytes, "kernels": {}}
        for name, fn in launches.items():
            for i in range(min(P, 4)):
                fn(i)
            torch.cuda.synchronize()
            reps = 2 * P
            fdl.fd_timer_arm(name, reps)
            for r in range(reps):
                fn(r % P)
            torch.cuda.synchronize()
            ms = fdl.fd_timer_read(reps)
            fdl.fd_timer_disarm()
            avg = float(np.mean(ms))
            nbytes = kernel_bytes(name, w, M)
            gbs = nbytes / (avg * 1e-3) / 1e9
            res["kernels"][name] = {"bytes": nbytes, "avg_us": avg * 1e3, "achieved": gbs, "peak": PEAK_HBM_GBS,
                                    "unit": "GB/s", "frac": gbs / PEAK_HBM_GBS, "launches": len(ms)}
        out[label] = res
        del xs, vs, vcs, xa
        torch.cuda.empty_cache()
    # reference: a plain device copy (torch) of 256 MiB per launch under the same
    # rotating-buffer rule, read + write bytes
    n = 64 << 20
    bufs = [torch.empty(n, device="cuda") for _ in range(10)]
    outs = [torch.empty(n, device="cuda") for _ in range(10)]
    outs[0].copy_(bufs[0])
    ts = []
    for i in range(10):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        outs[i].copy_(bufs[i])
        e1.record()
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1))
    t = float(np.median(ts))
    out["copy_reference"] = {"bytes": 8.0 * n, "avg_us": t * 1e3, "achieved": 8.0 * n / (t * 1e-3) / 1e9,
                             "unit": "GB/s", "frac": 8.0 * n / (t * 1e-3) / 1e9 / PEAK_HBM_GBS}
    del bufs, outs
    torch.cuda.empty_cache()
    return out


def step_flops(w, M: int) -> float:
    per_block = sum(kernel_flops(k, w, M) for k in ("gemm_qkv", "gemm_o", "gemm_mlp1", "gemm_mlp2", "attn"))
    return w.L * per_block + kernel_flops("embed", w, M) + kernel_flops("final", w, M)


KERNEL_SOURCES = {"attn": ("k_attn.hip", "fd_attn_sched.h", "fd_rules.h", "fd_common.h")}
for _g in ("gemm_qkv", "gemm_o", "gemm_mlp1", "gemm_mlp2"):
    KERNEL_SOURCES[_g] = ("k_gemm.hip", "fd_gemm_rules.h", "fd_rules.h", "fd_common.h")


def traffic_per_launch(kernel: str, workload: str):
    """HBM bytes per launch from the committed counter summary of this kernel and
    workload, or None if there is none or the kernel's sources changed since."""
    from paper_2607_12121_amd.rocprof_summary import read_traffic
    srcs = [os.path.join(ROOT, "paper_2607_12121_amd", "csrc", f) for f in KERNEL_SOURCES.get(kernel, ())]
    if not srcs:
        return None
    return read_traffic(os.path.join(ROOT, "profiles", f"{kernel}_{workload}_traffic.txt"), srcs)


def cpu_baseline(w, params_gpu, M_expected: int, budget_s: float, max_rows: int = 1024, threads=None):
    """The oracle on the host cores, on a bounded sample of one step of the same
    workload: the gate and embedding of all rows, then DiT blocks run on a
    sample of at most `max_rows` of the active rows (their keys and values
    written to the cache, their queries attending to every token of the
    request, their MLP) for as many blocks as fit the budget, then the final
    layer and update of all rows.  Every per-block cost of the oracle is linear
    in the rows it runs, so the step time is extrapolated as the sampled block
    time x (active rows / sampled rows) x L.  threads: cap on the BLAS threads
    (None: as many as the host gives)."""
    from threadpoolctl import threadpool_limits

    if threads is not None:
        with threadpool_limits(limits=threads):
            r = cpu_baseline(w, params_gpu, M_expected, budget_s, max_rows)
        r["cores"] = min(r["cores"], threads)
        return r
    import torch
    from threadpoolctl import threadpool_info

    from oracle import flashdiff_oracle as orc
    from paper_2607_12121_amd import workloads as wl

    rm = wl.region_map(w)
    lay = orc.Layout(rm.token_region.astype(np.int64), rm.req_tok_off.astype(np.int64), rm.n_regions)
    inp = wl.step_inputs(w, 0, rmap=rm)
    cond = wl.make_cond(w).numpy().astype(np.float64)
    p64 = {k: params_gpu[k].to("cpu", torch.float64).numpy()
           for k in ("w_e", "b_e", "pos", "w_adaf", "b_adaf", "w_out", "b_out")}
    t0 = time.perf_counter()
    score = orc.region_score(lay, inp.x_cur, inp.x_prev)
    st, run, act = orc.gate_select(lay, score, np.zeros(w.R), np.zeros(w.R, np.int32), np.ones(w.R, bool),
                                   inp.eps, 0.0, 0)
    idx, cu = orc.active_rows(lay, act)
    treq = lay.token_request()[idx]
    h = orc.embed(inp.x_cur[idx].astype(np.float64), idx, p64["w_e"], p64["b_e"], p64["pos"])
    t_gate = time.perf_counter() - t0
    M = len(idx)
    rng = np.random.default_rng(0)
    sel = np.sort(rng.choice(M, min(M, max_rows), replace=False))
    hs = h[sel]
    blocks, t_blocks = 0, 0.0
    while blocks < w.L and (blocks < 1 or t_blocks < budget_s):
        blk = {k: params_gpu[k][blocks].to("cpu", torch.float64).numpy()
               for k in ("w_qkv", "b_qkv", "w_o", "b_o", "w_1", "b_1", "w_2", "b_2", "w_ada", "b_ada")}
        kc = rng.standard_normal((w.N, w.D))
        vc = rng.standard_normal((w.N, w.D))
        t1 = time.perf_counter()
        hs = orc.block_forward(hs, idx[sel], treq[sel], lay, blk, cond, kc, vc, w.H)
        t_blocks += time.perf_counter() - t1
        blocks += 1
    t2 = time.perf_counter()
    v = orc.final_layer(h, treq, p64["w_adaf"], p64["b_adaf"], p64["w_out"], p64["b_out"], cond)
    orc.latent_update(inp.x_cur, v, idx, lay, wl.dt_per_request(w), np.zeros((w.N, w.C), np.float32), act,
                      orc.FREEZE)
    t_tail = time.perf_counter() - t2
    t_step = t_gate + t_tail + t_blocks / blocks * (M / len(sel)) * w.L
    # the oracle's parallelism is its BLAS library's thread pool
    threads = max([i.get("num_threads", 1) for i in threadpool_info() if i.get("user_api") == "blas"] + [1])
    return {"value": M / t_step, "unit": "active tokens/s", "cores": int(threads), "kind": "oracle",
            "sample": f"one {w.name} step (M={M} active rows): gate + embed of all rows, {blocks} of {w.L} DiT "
                      f"blocks on {len(sel)} sampled active rows (scaled by {M / len(sel):.2f} rows and to {w.L} "
                      f"blocks), final + update of all rows; {t_gate + t_blocks + t_tail:.1f} s of CPU work; "
                      f"host nproc={os.cpu_count()}",
            "seconds_per_step": t_step, "host": {"nproc": os.cpu_count(), "cpu": _cpu_model()}}


def _cpu_model() -> str:
    """The host CPU's model name (first `model name` line of /proc/cpuinfo), or ""."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return ""


def trajectory_study(torch, fdl, wl, w, rm, params, kc, vc, plan, d, cond, dt, T: int,
                     cs=(0.9, 0.95, 1.0, 1.05, 1.1, 1.2)) -> dict:
    """Chained steps x_{n+1} = x_n + dt v(x_n) from the same start, one dense warm-up
    step (eps = 0) then T - 1 gated steps (stateful gate, forced reactivation after
    K = 5 skips), for thresholds eps_b = c / R_b and both skip modes; reports the
    final latent's normwise distance to the dense trajectory (eps = 0 throughout)
    and the mean active fraction.  Sec. 3.2 bounds that distance by
    O(eps * sum_n D_n + gamma)."""
    inp = wl.step_inputs(w, 0, rmap=rm)
    regs = np.diff(rm.req_reg_off).astype(np.float64)

    def run(c: float, mode: int):
        st = fdl.SparseStep(plan, d, params, w.L, k_cache=kc.clone(), v_cache=vc.clone())
        x = torch.from_numpy(inp.x_cur).cuda()
        xp = torch.from_numpy(inp.x_prev).cuda()
        act = []
        for n in range(T):
            eps = torch.from_numpy(np.zeros(w.B) if n == 0 else c / regs).cuda()
            x_old = x.clone()
            st.step(x, xp, eps, dt, cond, max_skip=5, skip_mode=mode)
            xp = x_old
            if n > 0:
                act.append(int(st.m.item()) / w.N)
        torch.cuda.synchronize()
        return x, float(np.mean(act)) if act else 1.0

    x_ref, _ = run(0.0, fdl.FD_SKIP_FREEZE)
    runs = []
    for mode, name in ((fdl.FD_SKIP_FREEZE, "freeze"), (fdl.FD_SKIP_REUSE_DRIFT, "reuse_drift")):
        for c in cs:
            x, af = run(c, mode)
            dev = float(torch.linalg.vector_norm(x - x_ref) / torch.linalg.vector_norm(x_ref))
            runs.append({"mode": name, "eps_times_regions": c, "active_frac": af, "rel_dev": dev})
    return {"trajectory": {"workload": w.name, "steps": T, "max_skip": 5, "dt": float(dt[0].item()), "runs": runs}}


def trajectory_for(torch, fdl, wl, name: str, T: int, **kw) -> dict:
    """trajectory_study on workload `name` with its synthetic weights and caches."""
    w = wl.WORKLOADS[name]
    rm = wl.region_map(w)
    params = wl.make_params(w, device="cuda")
    kc, vc = wl.make_kv_cache(w, device="cuda")
    plan = fdl.make_plan(rm.token_region, rm.req_tok_off, rm.n_regions)
    d = fdl.dims(w.C, w.D, w.H, w.dh, w.F)
    cond = wl.make_cond(w, device="cuda")
    dt = torch.from_numpy(wl.dt_per_request(w)).cuda()
    return trajectory_study(torch, fdl, wl, w, rm, params, kc, vc, plan, d, cond, dt, T, **kw)


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "the region-sparse step is implemented for a single GPU; use --gpus 1", "n_gpus": args.gpus}))
        return 2
    import torch

    from paper_2607_12121_amd import flashdiff as fdl
    from paper_2607_12121_amd import workloads as wl

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        return 2
    torch.cuda.set_device(0)
    if args.copy_probe_mib > 0:
        src = torch.ones(args.copy_probe_mib << 18, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.neg(src, out=dst)
        torch.cuda.synchronize()
        del src, dst
    if args.trajectory > 0:
        print(json.dumps(trajectory_for(torch, fdl, wl, args.workload, args.trajectory)), flush=True)
        return 0

    res = time_workload(torch, fdl, wl, args.workload, args.steps, args.warmup, args.pool)
    w, M = res["w"], res["M"]
    out = {
        "metric": "active tokens/sec per region-sparse DiT step; % bf16 MFMA peak",
        "value": res["value"],
        "unit": "active tokens/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": res["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": res["config"],
        "step_mfma_frac": res["step_mfma_frac"],
        "roofline": res["roofline"],
        "kernels_ms_per_step": res["kernels_ms_per_step"],
    }
    out["importance"] = importance_cost(fdl, res["stp"], res["run"], w, M, args.warmup + args.steps)
    params = res["params"]
    del res
    torch.cuda.empty_cache()
    if not args.no_secondary and args.workload != "image":
        print("[bench] secondary figure: the image workload", file=sys.stderr, flush=True)
        sec = time_workload(torch, fdl, wl, "image", args.steps, args.warmup, args.pool)
        out["secondary"] = {k: sec[k] for k in ("value", "unit", "ms_per_step", "config", "step_mfma_frac",
                                                "roofline", "kernels_ms_per_step")}
        del sec
        torch.cuda.empty_cache()
    if not (args.no_trajectory or args.no_secondary) and args.workload != "image":
        # the chained-trajectory study at two thresholds around the designed gap (with
        # the secondary figures: runs that skip those, e.g. the profiled ones, skip it)
        print("[bench] trajectory study: image, 50 chained steps", file=sys.stderr, flush=True)
        out["trajectory"] = trajectory_for(torch, fdl, wl, "image", 50, cs=(1.0, 1.05))["trajectory"]
        torch.cuda.empty_cache()
    out["partition"] = partition_cost(torch, fdl, wl)
    if not args.no_hbm:
        print("[bench] streaming-kernel bandwidth (score, gather, scatter)", file=sys.stderr, flush=True)
        out["hbm"] = hbm_streams(torch, fdl, wl)
    if not args.no_cpu_baseline:
        print("[bench] timing the CPU oracle sample", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(w, params, M, args.cpu_seconds, threads=args.cpu_threads)
    print(json.dumps(out), flush=True)
    return 0


def time_workload(torch, fdl, wl, name: str, steps: int, warmup: int, pool: int) -> dict:
    """Times `steps` region-sparse steps of workload `name` (inputs resident in HBM,
    stateless gate at the designed thresholds) and the dominant MFMA kernel's
    launches inside them; returns the figures and the objects used."""
    w = wl.WORKLOADS[name]
    rm = wl.region_map(w)
    print(f"[bench] workload {w.name}: N={w.N} R={w.R} D={w.D} L={w.L}; drawing inputs on the GPU",
          file=sys.stderr, flush=True)
    params = wl.make_params(w, device="cuda")
    kc, vc = wl.make_kv_cache(w, device="cuda")
    plan = fdl.make_plan(rm.token_region, rm.req_tok_off, rm.n_regions)
    d = fdl.dims(w.C, w.D, w.H, w.dh, w.F)
    stp = fdl.SparseStep(plan, d, params, w.L, k_cache=kc, v_cache=vc)
    pairs, expected_m = [], []
    for i in range(pool):
        inp = wl.step_inputs(w, i, rmap=rm)
        pairs.append((torch.from_numpy(inp.x_cur).cuda(), torch.from_numpy(inp.x_prev).cuda(),
                      torch.from_numpy(inp.eps).cuda()))
        expected_m.append(int(inp.hot[rm.token_region].sum()))
    cond = wl.make_cond(w, device="cuda")
    dt = torch.from_numpy(wl.dt_per_request(w)).cuda()

    def run(i):
        x, xp, eps = pairs[i % pool]
        stp.step(x, xp, eps, dt, cond, stateless=True)

    for i in range(warmup):
        run(i)
    torch.cuda.synchronize()

    # per-kernel time per step (untimed calibration pass, one kernel type at a time)
    per_kernel = {}
    for kname in (k for k in fdl.KERNELS if k not in ("importance", "partition")):
        fdl.fd_timer_arm(kname, 4 * w.L + 8)
        run(0)
        torch.cuda.synchronize()
        ms = fdl.fd_timer_read(4 * w.L + 8)
        fdl.fd_timer_disarm()
        per_kernel[kname] = (float(ms.sum()), len(ms))
    mfma_kernels = ("gemm_qkv", "gemm_o", "gemm_mlp1", "gemm_mlp2", "attn")
    dominant = max(mfma_kernels, key=lambda k: per_kernel[k][0])

    # timed region: K steps, the dominant kernel's launches bracketed by HIP events
    cap = steps * 2 * w.L + 8
    fdl.fd_timer_arm(dominant, cap)
    torch.cuda.synchronize()
    t_start = torch.cuda.Event(enable_timing=True)
    t_end = torch.cuda.Event(enable_timing=True)
    t_start.record()
    for i in range(steps):
        run(warmup + i)
    t_end.record()
    torch.cuda.synchronize()
    ms_total = t_start.elapsed_time(t_end)
    dom_ms = fdl.fd_timer_read(cap)
    fdl.fd_timer_disarm()
    M = int(stp.m.item())
    last = (warmup + steps - 1) % pool
    assert M == expected_m[last], f"active rows {M} != designed {expected_m[last]}"
    m_mean = float(np.mean([expected_m[(warmup + i) % pool] for i in range(steps)]))
    ms_step = ms_total / steps
    dom_avg_ms = float(np.mean(dom_ms))
    achieved = kernel_flops(dominant, w, M) / (dom_avg_ms * 1e-3) / 1e12
    print(f"[bench] {w.name}: {ms_step:.3f} ms/step, {dominant} {dom_avg_ms * 1e3:.1f} us/launch",
          file=sys.stderr, flush=True)
    return {
        "w": w, "M": M, "stp": stp, "run": run, "params": params,
        "value": m_mean / (ms_step * 1e-3), "unit": "active tokens/s", "ms_per_step": ms_step,
        "config": {"workload": w.description, "tokens": w.N, "active_tokens": m_mean, "regions": w.R,
                   "active_regions": m_mean * w.R / w.N, "blocks": w.L, "hidden": w.D, "heads": w.H,
                   "head_dim": w.dh, "mlp": w.F, "latent_channels": w.C,
                   "gate": "stateless, eps at the designed gap", "parallelism": "single GPU"},
        "step_mfma_frac": step_flops(w, M) / (ms_step * 1e-3) / (PEAK_BF16_TFLOPS * 1e12),
        "roofline": {"kernel": dominant, "bound": "mfma", "achieved": achieved, "peak": PEAK_BF16_TFLOPS,
                     "unit": "TFLOP/s", "frac": achieved / PEAK_BF16_TFLOPS,
                     "traffic": traffic_per_launch(dominant, w.name), "launches": len(dom_ms),
                     "avg_ms": dom_avg_ms},
        "kernels_ms_per_step": {k: round(v[0], 4) for k, v in per_kernel.items()},
    }


if __name__ == "__main__":
    sys.exit(main())
