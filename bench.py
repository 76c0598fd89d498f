#!/usr/bin/env python3
"""Benchmark of the token-wise attention hot path on one MI355X.

A step is one pass of the whole path over one batch of synthetic inputs already resident in HBM:
score -> top-k -> refresh of the selected K/V cache rows -> attention of the selected queries over the
full-length K/V -> scatter into the cached outputs.  Prints ONE JSON line.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg3] [--budget PCT]
    python bench.py --sweep            # config 4: per-step time against a drawn budget schedule
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time
from pathlib import Path

ROOT = Path(__file__).resolve().parent
if str(ROOT) not in sys.path:
    sys.path.insert(0, str(ROOT))

METRIC = "selected-token attn TFLOP/s (% MFMA peak) + ms/layer, N=118800 H=24 D=128"
# MI355X dense MFMA peaks; an fp32 product is six products of bf16 parts
PEAK_TFLOPS = {"bf16": 2500.0, "f32": 2500.0 / 6}
PEAK_HBM_GBS = 8000.0
TRAFFIC_PROFILE = ROOT / "profiles" / "hot_path_cfg3_hbm_traffic_and_mfma.txt"
_CSRC = ROOT / "paper_2506_05096_amd" / "csrc"
KERNEL_SOURCE = {"attn_bf16_kernel": (_CSRC / "attn_bf16.hip", _CSRC / "gfx950.h")}


def kernel_source_hash(kernel: str) -> str:
    """First 16 hex digits of the SHA-256 of the kernel's source files, in the order listed above."""
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCE[kernel]:
        h.update(f.read_bytes())
    return h.hexdigest()[:16]


def measured_traffic(kernel: str, workload: str, budget: int):
    """HBM bytes one launch of the dominant kernel moves, as the tracked rocprofv3 summary recorded them
    (FETCH_SIZE + WRITE_SIZE, each scaled by what the same counter reads for the library's plain 1 GiB copy).
    The summary carries a line
        roofline_traffic kernel=<name> workload=<cfg> budget_pct=<p> fetched_bytes=<f> written_bytes=<w> source_sha256_16=<h>
    where <h> is kernel_source_hash() of the kernel's source files at the time of the profile.  Returns (bytes, note); bytes is
    None when there is no line for this workload or when the kernel source has changed since (a stale figure
    would say nothing about the kernel being timed)."""
    import re
    if not TRAFFIC_PROFILE.exists() or kernel not in KERNEL_SOURCE:
        return None, "no counter profile for this kernel"
    now = kernel_source_hash(kernel)
    for line in TRAFFIC_PROFILE.read_text().splitlines():
        m = re.search(r"roofline_traffic kernel=(\S+) workload=(\S+) budget_pct=(\d+) fetched_bytes=(\S+) "
                      r"written_bytes=(\S+) source_sha256_16=(\S+)", line)
        if m and m.group(1) == kernel and m.group(2) == workload and int(m.group(3)) == budget:
            if m.group(6) != now:
                return None, (f"{TRAFFIC_PROFILE.name} was recorded for another version of {KERNEL_SOURCE[kernel][0].name} "
                              f"({m.group(6)}, now {now}): rerun the FETCH_SIZE / WRITE_SIZE passes")
            return float(m.group(4)) + float(m.group(5)), f"read from profiles/{TRAFFIC_PROFILE.name} (kernel source {now})"
    return None, f"profiles/{TRAFFIC_PROFILE.name} has no counters for {workload} at {budget} %"


def budget_sweep(torch, layer, t, levels=tuple(range(10, 101, 10)), reps=2):
    """Config 4 in short, inside the default run: `reps` timed layer-steps at every budget level on the resident
    inputs, and how far the per-step time is from a line through the origin (the paper's "latency increases
    linearly with the computation budget").  bench.py --sweep runs the drawn 50-step schedule with fresh inputs."""
    import numpy as np
    ms = {}
    for pct in levels:
        k = layer.budget_to_k(pct)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(reps):
            layer.run(t, k)
        b.record()
        torch.cuda.synchronize()
        ms[pct] = a.elapsed_time(b) / reps
    x = np.array(sorted(ms), float)
    y = np.array([ms[int(p)] for p in x], float)
    slope = float((x * y).sum() / (x * x).sum())            # least-squares line through the origin
    dev = np.abs(y - slope * x) / (slope * x)
    return {"ms_by_budget": {str(int(p)): float(v) for p, v in zip(x, y)}, "ms_per_percent": slope,
            "max_rel_dev_from_linear": float(dev.max()), "at_budget_pct": int(x[int(dev.argmax())]),
            "mean_rel_dev_from_linear": float(dev.mean()), "dense_step_ms": float(y[-1]),
            "steps_per_level": reps,
            "what": "whole layer-step (score + top-k + K/V refresh + attention + scatter) at each budget level, "
                    "deviation from the least-squares line through the origin"}


def _np(t):
    import numpy as np
    import torch
    t = t.detach().cpu().contiguous()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def cpu_baseline(w, t, idx_sel_host, k, scale, target_s=15.0):
    """The CPU oracle, as it stands, on a bounded sample of the same workload: score and top-k in full,
    attention and scatter on the first `rows` selected tokens (all heads, all N keys)."""
    import numpy as np
    import oracle
    n, H, D = w.N, w.H, w.D
    xc, xp = _np(t["x_cur"]), _np(t["x_prev"])
    kc, vc, q = _np(t["k_cache"]), _np(t["v_cache"]), _np(t["q"])
    cache = _np(t["out_cache"]).copy()
    t0 = time.perf_counter()
    sc = oracle.score(xc, xp)
    idx, _, _ = oracle.topk(sc, k)
    t_sel = time.perf_counter() - t0
    # calibrate on 2 rows, then size the sample for ~target_s
    t0 = time.perf_counter()
    oracle.sparse_attn(q, kc, vc, idx[:2], scale)
    per_row = max((time.perf_counter() - t0) / 2, 1e-6)
    rows = int(max(2, min(k, target_s / per_row)))
    t0 = time.perf_counter()
    o64, _ = oracle.sparse_attn(q, kc, vc, idx[:rows], scale)
    o = oracle.round_to_dtype(o64.reshape(rows, H * D), oracle.BF16 if w.dtype == "bf16" else oracle.F32)
    oracle.scatter(cache, o, idx[:rows])
    t_attn = time.perf_counter() - t0
    flops = 4.0 * rows * n * D * H
    return {
        "value": flops / (t_sel * rows / max(k, 1) + t_attn) / 1e12,
        "unit": "TFLOP/s",
        "cores": oracle.num_threads(),
        "kind": "oracle",
        "sample": f"score+top-k on all {n} tokens ({t_sel:.2f} s, charged pro rata), attention+scatter on the first "
                  f"{rows} of {k} selected tokens x {H} heads x {n} keys ({t_attn:.2f} s, fp64 accumulation)",
        "indices_match_gpu": bool(np.array_equal(idx, idx_sel_host)),
    }


def measured_peaks(torch, ab, copy_reps=2):
    """What this chip sustains on the two resources the path leans on, measured with the library's probes:
    a register-resident bf16 MFMA loop (constant and pseudo-random operands; random data runs into the
    power limit) and a plain 1 GiB device copy."""
    dev = "cuda:0"
    ev = lambda: torch.cuda.Event(enable_timing=True)
    out = {}
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sink = torch.empty(cus * 2 * 256, device=dev)
    for name, rnd in (("mfma_bf16_const_TFLOPs", False), ("mfma_bf16_random_TFLOPs", True)):
        ab.astraea_probe_mfma_bf16(cus * 2, 20000, rnd, sink)
        a, b = ev(), ev()
        a.record()
        fl = ab.astraea_probe_mfma_bf16(cus * 2, 400000, rnd, sink)      # ~50 ms: long enough for clocks to settle
        b.record()
        torch.cuda.synchronize()
        out[name] = fl / a.elapsed_time(b) / 1e9
    n = 1 << 30
    src = torch.empty(n, dtype=torch.uint8, device=dev).fill_(1)
    dst = torch.empty(n, dtype=torch.uint8, device=dev)
    ab.astraea_probe_copy(src, dst)
    a, b = ev(), ev()
    a.record()
    for _ in range(copy_reps):
        ab.astraea_probe_copy(src, dst)
    b.record()
    torch.cuda.synchronize()
    out["copy_read_plus_write_GBps"] = 2.0 * n * copy_reps / a.elapsed_time(b) / 1e6
    out["copy_bytes_each_way"] = n
    return out


def library_context(torch, w, k):
    """Context only, same GPU and shape: the vendor libraries PyTorch dispatches to (a bf16 GEMM and the
    library flash attention) on dense tensors of the workload's shape.  Not part of the path."""
    dev = "cuda:0"
    ev = lambda: torch.cuda.Event(enable_timing=True)
    out = {}
    n = 8192
    a = torch.randn(n, n, device=dev).bfloat16()
    b = torch.randn(n, n, device=dev).bfloat16()
    for _ in range(3):
        a @ b
    e0, e1 = ev(), ev()
    e0.record()
    for _ in range(20):
        a @ b
    e1.record()
    torch.cuda.synchronize()
    out["torch_matmul_bf16_8192_TFLOPs"] = 2.0 * n ** 3 / (e0.elapsed_time(e1) / 20) / 1e9
    del a, b
    if w.dtype == "bf16":
        q = torch.randn(1, w.H, k, w.D, device=dev).bfloat16()
        kk = torch.randn(1, w.H, w.N, w.D, device=dev).bfloat16()
        vv = torch.randn(1, w.H, w.N, w.D, device=dev).bfloat16()
        sdpa = torch.nn.functional.scaled_dot_product_attention
        for _ in range(2):
            sdpa(q, kk, vv)
        e0, e1 = ev(), ev()
        e0.record()
        for _ in range(3):
            sdpa(q, kk, vv)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / 3
        out["torch_sdpa_bf16_same_shape_ms"] = ms
        out["torch_sdpa_bf16_same_shape_TFLOPs"] = 4.0 * k * w.N * w.D * w.H / ms / 1e9
    return out


def token_sparse_block(torch, ab, w, t, k, reps=5):
    """The per-token layers of a block on the k selected rows (Q/K/V and output projections, two MLP layers, each
    one astraea_sparse_linear call with synthetic bf16 weights) and the whole block step with them.  Reported
    beside the headline; the flops are 2*k*c_in*c_out per layer (the projection and MLP terms of the paper's FLOPs
    appendix with N -> k)."""
    from paper_2506_05096_amd.layer import TokenSparseBlock
    E, hid, dev = w.H * w.D, 4 * w.H * w.D, t["q"].device
    g = torch.Generator(device=dev).manual_seed(4242)
    mk = lambda o, i: (torch.randn(o, i, device=dev, generator=g) * i ** -0.5).bfloat16()
    weights = {"wqkv": mk(3 * E, E), "wo": mk(E, E), "w1": mk(hid, E), "w2": mk(E, hid),
               "b1": torch.zeros(hid, dtype=torch.bfloat16, device=dev), "b2": torch.zeros(E, dtype=torch.bfloat16, device=dev)}
    blk = TokenSparseBlock(w.N, w.H, w.D, weights, device=dev)
    # packed [N, 3, H, D] cache: Q, K and V of a token side by side, written by one stacked projection
    tt = {"x_in": t["x_cur"], "x_prev": t["x_prev"], "out_cache": t["out_cache"],
          "qkv_cache": torch.stack([t["q"], t["k_cache"], t["v_cache"]], dim=1).contiguous()}
    if tt["x_in"].shape[1] != E:
        return {"skipped": "feature width of this workload is not H*D"}
    blk.run(tt, k)
    torch.cuda.synchronize()
    ev = lambda: torch.cuda.Event(enable_timing=True)
    parts = {"qkv_proj": lambda: blk.step_qkv(tt, k), "attn": lambda: blk.step_attn(tt, k),
             "out_proj_mlp": lambda: blk.step_proj_mlp(tt, k)}
    ms = {}
    for nm, fn in parts.items():
        a, b = ev(), ev()
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        torch.cuda.synchronize()
        ms[nm] = a.elapsed_time(b) / reps
    t0 = time.perf_counter()
    for _ in range(reps):
        blk.run(tt, k)
    torch.cuda.synchronize()
    step_ms = (time.perf_counter() - t0) * 1e3 / reps
    fl = blk.flops(k)
    fl_qkv, fl_rest = fl["qkv_proj"], fl["out_proj"] + fl["mlp"]
    lin_ms = ms["qkv_proj"] + ms["out_proj_mlp"]
    return {"ms_per_step": step_ms, "ms": ms,
            "linear_TFLOPs": (fl_qkv + fl_rest) / lin_ms / 1e9,
            "linear_frac_of_mfma_peak": (fl_qkv + fl_rest) / lin_ms / 1e9 / PEAK_TFLOPS["bf16"],
            "linear_flops": fl_qkv + fl_rest,
            "what": "score + top-k + stacked Q/K/V projection of the selected rows written into a packed cache + "
                    "attention + output projection + 2 MLP layers (the last writes the cached block output); "
                    "hidden width 4*H*D"}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="cfg3")
    ap.add_argument("--budget", type=int, default=None, help="token budget in percent (default: the workload's)")
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--sweep", action="store_true", help="config 4: 50-step budget schedule")
    ap.add_argument("--context", action="store_true",
                    help="also time the vendor-library GEMM and flash attention PyTorch dispatches to (context only)")
    ap.add_argument("--source-hash", action="store_true",
                    help="print the hash of the dominant kernel's sources that a counter profile must carry, and exit")
    ap.add_argument("--calibrate", action="store_true",
                    help="only run the measurement aids: 1 GiB plain copy (x3) and the MFMA loop")
    args = ap.parse_args()
    if args.source_hash:
        print(kernel_source_hash("attn_bf16_kernel"))
        return 0
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on exactly one GPU (no collectives, no sharding); use --gpus 1",
              file=sys.stderr)
        return 2

    import torch
    from paper_2506_05096_amd import binding as ab
    from paper_2506_05096_amd import synth
    from paper_2506_05096_amd.build import ensure_built
    from paper_2506_05096_amd.layer import LayerStep

    ensure_built()
    ab.lib()
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    torch.cuda.set_device(0)
    w = synth.WORKLOADS[args.workload]
    if args.calibrate:
        print(json.dumps(measured_peaks(torch, ab, copy_reps=3)))
        return 0
    if args.sweep:
        return sweep(args, w if args.workload == "cfg4" else synth.WORKLOADS["cfg4"])
    budget = args.budget if args.budget is not None else w.budgets_pct[0]
    t = synth.make_layer_inputs(w, seed=args.seed, device=dev)
    layer = LayerStep(w.N, w.H, w.D, w.torch_dtype, device=dev)
    k = layer.budget_to_k(budget)
    es = 2 if w.dtype == "bf16" else 4

    ev = lambda: torch.cuda.Event(enable_timing=True)
    for _ in range(args.warmup):
        layer.run(t, k)
    torch.cuda.synchronize()
    attn_ev = [(ev(), ev()) for _ in range(args.steps)]
    ab.kernel_timer(True)          # the library brackets the attention's main kernel with HIP events on its stream
    t0 = time.perf_counter()
    for s in range(args.steps):
        layer.step_score(t)
        layer.step_select(k)
        layer.step_kv_refresh(t, k)
        attn_ev[s][0].record()
        layer.step_attn(t, k)
        attn_ev[s][1].record()
        layer.step_scatter(t, k)
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3 / args.steps
    attn_ms = sum(a.elapsed_time(b) for a, b in attn_ev) / args.steps       # the whole call
    kt = ab.kernel_times_ms()[:args.steps]
    ab.kernel_timer(False)
    idx_host = layer.idx_sel[:k].cpu().numpy()      # the timed steps' selection (later passes run other budgets)
    kernel_ms = sum(kt) / len(kt)                                           # its dominant kernel alone

    # untimed second pass: per-call durations for the breakdown
    names = ["score", "select_topk", "kv_refresh", "attn", "scatter"]
    calls = [lambda: layer.step_score(t), lambda: layer.step_select(k), lambda: layer.step_kv_refresh(t, k),
             lambda: layer.step_attn(t, k), lambda: layer.step_scatter(t, k)]
    reps = max(3, min(args.steps, 10))
    br = {}
    for nm, fn in zip(names, calls):
        a, b = ev(), ev()
        fn()
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        torch.cuda.synchronize()
        br[nm] = a.elapsed_time(b) / reps

    # the same step with the cache merge fused into the attention's last stage (one call fewer, no compact
    # result): reported beside the headline, which keeps every step of the path a call of its own
    fused = LayerStep(w.N, w.H, w.D, w.torch_dtype, device=dev, fused_update=True)
    fused.run(t, k)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(reps):
        fused.run(t, k)
    torch.cuda.synchronize()
    fused_ms = (time.perf_counter() - t1) * 1e3 / reps
    del fused

    flops = ab.astraea_attn_flops(w.N, k, w.H, w.D)
    row_bytes = w.H * w.D * es
    gbs = {
        "score": (2 * w.C * es + 4) * w.N / br["score"] / 1e6,
        "select_topk": (4 * 4 * w.N + 4 * k) / br["select_topk"] / 1e6,       # 3 radix passes + count, + indices
        "kv_refresh": 2 * 2 * row_bytes * k / br["kv_refresh"] / 1e6,
        "scatter": 2 * row_bytes * k / br["scatter"] / 1e6,
    }
    peak = PEAK_TFLOPS[w.dtype]
    achieved = flops / kernel_ms / 1e9
    kernel_name = "attn_bf16_kernel" if w.dtype == "bf16" else "attn_f32_kernel"
    traffic, traffic_note = measured_traffic(kernel_name, w.name, budget)
    out = {
        "metric": METRIC,
        "value": flops / wall_ms / 1e9,
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall_ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": "synthetic",
        "config": {"workload": f"{w.name}: N={w.N} H={w.H} D={w.D} C={w.C} budget={budget}% k={k} "
                               f"latent={'x'.join(map(str, w.latent))}",
                   "value_definition": "4*k*N*D*H flops / ms_per_step (whole hot path)", "seed": args.seed},
        "roofline": {"bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                     "frac": achieved / peak, "traffic": traffic, "traffic_source": traffic_note,
                     "traffic_unit": "bytes per launch (algorithmic: (2k+2N)*H*D*2 = %.3g)" % ((2 * k + 2 * w.N) * row_bytes),
                     "kernel": kernel_name,
                     "kernel_ms": kernel_ms, "call_ms": attn_ms, "flops_per_launch": flops,
                     "timed": "HIP events recorded by the library on the launch stream around the kernel alone, "
                              "mean over the timed steps; call_ms = the whole astraea_sparse_attn_fwd call "
                              "(for bf16 also the V re-tiling pre-pass and the partial-result merge)"},
        "breakdown_ms": br,
        "fused_update": {"ms_per_step": fused_ms, "value": flops / fused_ms / 1e9,
                         "what": "score + top-k + K/V refresh + astraea_sparse_attn_update_fwd"},
        "hbm_GBps": gbs,
        "hbm_frac_of_8TBps": {k_: v_ / PEAK_HBM_GBS for k_, v_ in gbs.items()},
    }
    if w.name in ("cfg3", "cfg4"):
        out["budget_sweep"] = budget_sweep(torch, layer, t)
    if w.dtype == "bf16" and w.D == 128:
        out["token_sparse_block"] = token_sparse_block(torch, ab, w, t, k)
    out["measured_peaks"] = measured_peaks(torch, ab)
    if w.dtype == "bf16":
        # the same box's register-resident MFMA loop on random operands: what the chip sustains under its power
        # limit with nothing but MFMAs; the sustained clock, and with it both figures, differs from box to box
        out["roofline"]["achieved_over_this_box_mfma_loop"] = achieved / out["measured_peaks"]["mfma_bf16_random_TFLOPs"]
    if args.context:
        out["library_context_same_gpu"] = library_context(torch, w, k)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, t, idx_host, k, layer.scale, args.cpu_seconds)
    print(json.dumps(out))
    return 0


def sweep(args, w) -> int:
    """Config 4: fresh tensors per step, budgets drawn from the seed; per-step ms against budget."""
    import numpy as np
    import torch
    from paper_2506_05096_amd import synth
    from paper_2506_05096_amd.layer import LayerStep
    dev = "cuda:0"
    sched = synth.budget_schedule(args.seed, 50)
    layer = LayerStep(w.N, w.H, w.D, w.torch_dtype, device=dev)
    t = synth.make_layer_inputs(w, seed=args.seed, device=dev, step=0)
    layer.run(t, layer.budget_to_k(100))           # warm-up (also the dense reference shape)
    torch.cuda.synchronize()
    rows = []
    for s, pct in enumerate(sched):
        fresh = synth.make_layer_inputs(w, seed=args.seed, device=dev, step=s + 1)
        for name in ("x_prev", "x_cur", "q", "k_new", "v_new"):
            t[name] = fresh[name]                  # caches (K, V, outputs) are carried across steps
        del fresh
        k = layer.budget_to_k(pct)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        layer.run(t, k)
        b.record()
        torch.cuda.synchronize()
        rows.append((pct, a.elapsed_time(b)))
        print(f"step {s:2d} budget {pct:3d}% k={k:6d} {rows[-1][1]:8.3f} ms", file=sys.stderr, flush=True)
    x = np.array([r[0] for r in rows], float)
    y = np.array([r[1] for r in rows], float)
    slope = float((x * y).sum() / (x * x).sum())            # least-squares line through the origin
    dev_rel = np.abs(y - slope * x) / (slope * x)
    dense = float(np.mean(y[x == 100])) if np.any(x == 100) else slope * 100
    by_budget = {int(p): float(np.mean(y[x == p])) for p in sorted(set(x))}
    print(json.dumps({
        "metric": "config-4 budget sweep: ms per layer-step vs token budget",
        "workload": f"cfg4: N={w.N} H={w.H} D={w.D}, 50 steps, budgets ~ U{{10..100%}}",
        "ms_by_budget": by_budget, "ms_per_percent": slope,
        "max_rel_dev_from_linear": float(dev_rel.max()), "mean_rel_dev_from_linear": float(dev_rel.mean()),
        "total_ms": float(y.sum()), "dense_step_ms": dense, "total_vs_50_dense": float(y.sum() / (50 * dense)),
        "mean_budget_pct": float(x.mean()),
    }))
    return 0


if __name__ == "__main__":
    sys.exit(main())
