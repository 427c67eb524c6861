#!/usr/bin/env python3
"""Benchmark of the expert-slot-cache MoE layer on one MI355X.

Workload (default): the A3B-shaped Q8_0 decode stack -- 48 MoE layers, hidden
2048, 128 experts, top-8, expert intermediate 768, weights N(0, 0.02)
quantised to Q8_0, fp32 router N(0, 0.05), 96 tokens decoded one at a time
with AR(1) hidden states (rho 0.8), 19 slots per layer (15%), LRU, the whole
28.7 GiB expert store in pinned host memory.  Data are synthetic and seeded.

One step = one full 96-token x 48-layer decode from a cold cache (every
layer's slot table reset), the layers chained h <- h + moe(rmsnorm(h)) on the
GPU (the library's residual and pre-norm flags).  --workload a3b_verify: the
same 96 tokens generated by speculative verification windows of 1 + 4 tokens
(one multi-token layer call per window and layer, seeded draft outcomes),
reported next to batch-1 decode on the same 25 % budget.
value = decoded tokens / wall seconds over the timed steps, inputs already in
HBM / pinned memory when timing starts.

Printed: one JSON line with the contract fields plus
  roofline      the dominant kernel of the step, from HIP events stamped at
                its launches in the timed region: for decode the fused
                copy + gate/up launch, bound by the host link (its algorithmic
                bytes are the misses' payloads; peak = PCIe 5.0 x16, one
                direction); with --copy-mode split the gate/up GEMV against the
                8 TB/s HBM peak; for prefill the copy kernel against the link,
                and with --warm (every expert resident, no copies) the gate/up
                grouped GEMM against the dense bf16 matrix peak;
  cpu_baseline  the CPU oracle on a bounded sample of the same workload;
  extra         hit rate, materialised bytes/token, copy GB/s vs the measured
                host-to-device peak, per-kernel timings.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# PCIe 5.0 x16, one direction: 32 GT/s x 16 lanes x 128/130 encoding / 8 bits
PCIE_PEAK_GBS = 32.0 * 16 * 128 / 130 / 8
BF16_PEAK_TFLOPS = 2500.0  # MI355X dense bf16 MFMA
HBM_BYTES = 288 * 10**9    # MI355X HBM3E capacity


def verify_windows(n_tokens, horizon, passes):
    """Speculative verification steps that generate n_tokens: each step verifies the window
    start .. start + horizon, keeps the longest run of passing drafts plus the target's own
    next token, and the next window starts after them.  Returns (start, accepted, generated)."""
    steps, start = [], 0
    while start < n_tokens:
        row = passes[len(steps)]
        accepted = 0
        while accepted < horizon and row[accepted]:
            accepted += 1
        made = min(accepted + 1, n_tokens - start)
        steps.append((start, accepted, made))
        start += made
    return steps


def kernel_sources_sha256_16():
    """Hash of every device source (csrc/*.hip and their headers, in name order): what a profile
    was measured on."""
    import hashlib
    csrc = os.path.join(ROOT, "paper_2607_09686_amd", "csrc")
    h = hashlib.sha256()
    for name in sorted(os.listdir(csrc)):
        if name.endswith((".hip", ".h")):
            h.update(name.encode() + b"\0")
            with open(os.path.join(csrc, name), "rb") as f:
                h.update(f.read() + b"\0")
    return h.hexdigest()[:16]


def measured_traffic(args, name, wl, budget):
    """Bytes per launch of a kernel from profiles/<name>_traffic.json, or None when the file is
    missing or was measured on other device sources, another workload, budget or policy."""
    path = os.path.join(args.profiles, name + "_traffic.json")
    if not os.path.exists(path) or budget != wl.budget_slots or args.policy != "lru":
        return None
    t = json.load(open(path))
    if t.get("kernel_sources_sha256_16") != kernel_sources_sha256_16() or t.get("workload") != wl.name:
        return None
    return t["traffic_bytes_per_launch"]


def log(msg):
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="a3b_decode",
                    choices=["a3b_decode", "a3b_sweep", "q4_decode", "q4km_decode", "tiny",
                             "a3b_prefill", "q4km_prefill", "a3b_verify"],
                    help="a3b_sweep: one cell of the cache-budget x locality sweep, chosen with "
                         "--budget (19, 45, 96) and --rho (0.3, 0.9)")
    ap.add_argument("--budget", type=int, default=None, help="slots per layer (default: workload's)")
    ap.add_argument("--warm", action="store_true",
                    help="keep the cache between steps instead of resetting it (with --budget equal "
                         "to the experts per layer, every expert stays resident after the warm-up: "
                         "a prefill step then runs its grouped GEMMs with no host copies beside them, "
                         "and the roofline is the gate/up GEMM against the bf16 matrix-core peak)")
    ap.add_argument("--rho", type=float, default=None)
    ap.add_argument("--no-timing", action="store_true", help="no HIP events around kernels")
    ap.add_argument("--timing-stride", type=int, default=16,
                    help="bracket one layer call in this many with HIP events")
    ap.add_argument("--copy-mode", default="kernel", choices=["kernel", "split", "side", "sdma"],
                    help="kernel: miss copies fused with gate/up in one launch (default); "
                         "split: copy kernel then gate/up kernel; side: hipMemcpyAsync on a "
                         "side stream overlapped with the hit experts; sdma: hipMemcpyAsync "
                         "on the compute stream")
    ap.add_argument("--cpu-sample-tokens", type=int, default=4)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--policy", default="lru", choices=["lru", "score"],
                    help="slot policy: lru (default, the workload's), or score: evict the resident "
                         "with the lowest router logit for the current token")
    ap.add_argument("--no-policy-bound", action="store_true",
                    help="skip the traced replay that bounds the misses from below (Belady MIN)")
    ap.add_argument("--profiles", default=os.path.join(ROOT, "profiles"),
                    help="directory of the measured bytes per launch (rocprofv3 --pmc) of the "
                         "roofline kernels; a file is used only if it was taken on the current "
                         "device sources and this workload")
    ap.add_argument("--hbm-probe", action="store_true",
                    help="decode: after the run, launch a plain HBM read of the down GEMV's bytes "
                         "per launch (256, 512 and 2048 blocks, 52 launches each) and an empty "
                         "launch, for a kernel trace that sets the GEMV against both on one clock")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="after the run, copy 256 MiB device-to-device 4 times with torch (a plain "
                         "copy kernel of known size, to scale the FETCH_SIZE / WRITE_SIZE counters)")
    return ap.parse_args()


def main():
    args = parse()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py measures one GPU only: the expert-slot-cache path has no multi-GPU "
              "mode (run with --gpus 1)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import synth
    from paper_2607_09686_amd import (KIND_COPY, KIND_DOWN, KIND_GATEUP, KIND_ROUTER, HostBuffer,
                                      MoeCache, min_misses, plan_percent, probe_h2d,
                                      probe_hbm_read)

    wl = synth.WORKLOADS[args.workload]
    # slots per layer from the workload's cache percentage, by the library's static planner;
    # the plan's lower bound (router weights + expert slots, no KV cache on this path) is
    # checked against the GPU's HBM
    model = {"n_layers": wl.n_layers, "n_experts": wl.n_experts, "top_k": wl.top_k,
             "payload_bytes": wl.payload_bytes, "common_bytes": wl.n_layers * wl.hidden * wl.n_experts * 4,
             "kv_bytes_per_token": 0, "overhead_bytes": 0, "target_bytes": HBM_BYTES}
    plan = plan_percent(model, wl.cache_percent)
    if plan["slots_per_layer"] != wl.budget_slots:
        raise RuntimeError(f"planner gives {plan['slots_per_layer']} slots, workload {wl.budget_slots}")
    budget = args.budget or wl.budget_slots
    rho = wl.rho if args.rho is None else args.rho
    if wl.sweep_slots and (budget not in wl.sweep_slots or rho not in wl.sweep_rhos):
        raise SystemExit(f"{wl.name}: choose --budget from {wl.sweep_slots} and --rho from {wl.sweep_rhos}")
    torch.cuda.set_device(0)

    log(f"workload {wl.name}: L={wl.n_layers} H={wl.hidden} E={wl.n_experts} k={wl.top_k} "
        f"I={wl.inter} {wl.qtype} C={budget} T={wl.n_tokens} rho={rho}")
    t0 = time.time()
    hb = HostBuffer(wl.store_bytes)
    log(f"pinned {wl.store_bytes / 2**30:.2f} GiB in {time.time() - t0:.1f} s")
    t0 = time.time()
    synth.expert_store(wl, out=hb.array)
    log(f"generated expert store in {time.time() - t0:.1f} s")
    R = synth.router(wl)
    verify = wl.mode == "verify"
    # verify windows reach horizon positions past the last generated token
    X = synth.hidden(wl, rho=rho, n_tokens=wl.n_tokens + (wl.horizon if verify else 0))
    Rd = torch.from_numpy(R).cuda()
    Xd = torch.from_numpy(X).cuda()
    windows = verify_windows(wl.n_tokens, wl.horizon,
                             synth.acceptance(wl.n_tokens, wl.horizon, wl.accept_q, wl.hidden_seed)) \
        if verify else None

    # measured pinned host-to-device bandwidth: 64 expert-sized copies, one stream
    # (the probe reads n_chunks * chunk bytes of the store: keep it inside the buffer)
    n_small = min(64, wl.store_bytes // wl.payload_bytes)
    h2d_peak = probe_h2d(hb.ptr, wl.payload_bytes, n_small, 1)
    h2d_big = probe_h2d(hb.ptr, 1 << 30, 4, 1) if wl.store_bytes >= 4 << 30 else None
    log(f"H2D probe: {h2d_peak:.1f} GB/s ({n_small} expert-size copies), {h2d_big} GB/s (1 GiB copies)")

    timing = not args.no_timing
    cache = MoeCache(wl.n_layers, wl.n_experts, wl.top_k, wl.hidden, wl.inter, wl.qtype, hb.ptr,
                     wl.store_bytes, budget, stream=torch.cuda.current_stream(), residual=True,
                     prenorm=True, timing=timing, copy_mode=args.copy_mode,
                     score_evict=args.policy == "score")
    if timing:
        cache.set_timing_stride(args.timing_stride)
    h = torch.empty(wl.hidden, dtype=torch.float32, device="cuda")
    y = torch.empty_like(h)

    prefill = wl.mode == "prefill"
    if prefill:
        h = torch.empty_like(Xd)
        y = torch.empty_like(Xd)
    W = wl.horizon + 1
    if verify:
        h = torch.empty((W, wl.hidden), dtype=torch.float32, device="cuda")
        y = torch.empty_like(h)

    def step(cache):
        nonlocal h, y
        if not args.warm:
            cache.reset()
        if prefill:  # the whole chunk through every layer
            h.copy_(Xd)
            for l in range(wl.n_layers):
                cache.layer_forward(h, Rd[l], l, y, n_tokens=wl.n_tokens)
                h, y = y, h
            return
        if verify:  # one window of 1 + horizon tokens through every layer per step
            for t, _, _ in windows:
                h.copy_(Xd[t:t + W])
                for l in range(wl.n_layers):
                    cache.layer_forward(h, Rd[l], l, y, n_tokens=W)
                    h, y = y, h
            return
        for t in range(wl.n_tokens):
            h.copy_(Xd[t])
            for l in range(wl.n_layers):
                cache.layer_forward(h, Rd[l], l, y, n_tokens=1)
                h, y = y, h

    kinds = ((KIND_ROUTER, "router"), (KIND_GATEUP, "gateup"), (KIND_DOWN, "down"),
             (KIND_COPY, "copy"))
    for i in range(args.warmup):
        step(cache)
        log(f"warmup step {i} done")
    torch.cuda.synchronize()
    counters = [0, 0, 0, 0]
    acc = {name: dict(launches=0, total_ms=0.0, bytes=0, flops=0) for _, name in kinds}
    def totals():
        """Counters and per-kind timing totals since the last reset (read before the next)."""
        st = {}
        if timing:
            for kind, name in kinds:
                s = cache.kernel_stats(kind)
                st[name] = (s.launches, s.total_ms, s.bytes, s.flops)
        return list(cache.counters().as_tuple()), st

    # with --warm the cache is not reset between steps: a step's share is the difference
    # of the totals around it
    base = totals() if args.warm else None
    ts = time.perf_counter()
    for i in range(args.steps):
        step(cache)
        now = totals()
        prev = base if args.warm else ([0, 0, 0, 0], {n: (0, 0.0, 0, 0) for n in now[1]})
        counters = [a + b - c for a, b, c in zip(counters, now[0], prev[0])]
        for name, (l, ms, b, f) in now[1].items():
            pl, pms, pb, pf = prev[1][name]
            a = acc[name]
            a["launches"] += l - pl
            a["total_ms"] += ms - pms
            a["bytes"] += b - pb
            a["flops"] += f - pf
        if args.warm:
            base = now
    torch.cuda.synchronize()
    dt = time.perf_counter() - ts
    log(f"timed {args.steps} steps in {dt:.2f} s")
    tokens = args.steps * wl.n_tokens
    hits, misses, evictions, mbytes = counters
    stats = {}
    for _, name in kinds:
        a = acc[name]
        if a["launches"]:
            stats[name] = dict(a, avg_us=1e3 * a["total_ms"] / a["launches"],
                               gb_per_s=a["bytes"] / (a["total_ms"] * 1e6) if a["total_ms"] else None)
    result = {
        "metric": ("MoE-layer prefill tokens/s; expert-FFN MFMA utilisation; materialized bytes/token"
                   if prefill else
                   "MoE-layer decode tokens/s; expert-FFN HBM GB/s; materialized bytes/token"),
        "value": tokens / dt,
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * dt / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16" if prefill else "f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "n_layers": wl.n_layers, "hidden": wl.hidden,
                   "n_experts": wl.n_experts, "top_k": wl.top_k, "inter": wl.inter,
                   "qtype": wl.qtype, "budget_slots": budget, "n_tokens": wl.n_tokens, "rho": rho,
                   "copy_mode": args.copy_mode, "policy": args.policy, "warm_cache": args.warm,
                   "global_batch": wl.n_tokens if prefill else 1, "seq_len": wl.n_tokens,
                   "parallelism": "none"},
    }
    if timing and prefill and "copy" not in stats:
        # a warm cache with every expert resident: no copies, the grouped GEMMs alone
        gu_st, dn_st = stats["gateup"], stats["down"]
        achieved = gu_st["flops"] / (gu_st["total_ms"] * 1e9)
        gu_name = ("pf_gateup_wide_kernel<%d>" if wl.inter % 128 == 0 and wl.hidden % 64 == 0 else
                   "gm_gateup_kernel<%d>" if wl.qcode in (12, 14) else "pf_gateup_kernel<%d>")
        result["roofline"] = {"bound": "mfma", "kernel": gu_name % (wl.qcode & 0xff),
                              "achieved": achieved, "peak": BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                              "frac": achieved / BF16_PEAK_TFLOPS, "traffic": None,
                              "avg_launch_us": 1e3 * gu_st["total_ms"] / max(1, gu_st["launches"]),
                              "note": "algorithmic flops 4 n H I per expert of n rows (the launch also "
                                      "multiplies the lo activation term: twice the MFMA work)"}
        ffn_ms = gu_st["total_ms"] + dn_st["total_ms"]
        ffn_bytes = gu_st["bytes"] + dn_st["bytes"]
    elif timing and (verify or prefill):
        # the misses are copied by the copy kernel while the MFMA GEMMs of earlier
        # experts run beside it: the copies dominate and the host link bounds them
        cp = stats["copy"]
        avg_s = cp["total_ms"] / 1e3 / max(1, cp["launches"])
        per_launch_bytes = cp["bytes"] / max(1, cp["launches"])
        achieved = cp["bytes"] / (cp["total_ms"] * 1e6)
        if not verify:
            kernel = "materialize_kernel"
        elif args.copy_mode == "kernel":
            kernel = "copy_gateup_mt_kernel<%d> (device work list; the union's gate/up inside)" % (
                8 if wl.qtype == "q8_0" else 2)
        else:
            kernel = "materialize_list_kernel (device work list)"
        result["roofline"] = {"bound": "pcie", "kernel": kernel, "achieved": achieved,
                              "peak": PCIE_PEAK_GBS, "unit": "GB/s", "frac": achieved / PCIE_PEAK_GBS,
                              "traffic": None, "bytes_per_copy": per_launch_bytes,
                              "avg_us_per_copy": avg_s * 1e6}
        none = {"total_ms": 0.0, "bytes": 0, "flops": 0}
        gu_st, dn_st = stats.get("gateup", none), stats.get("down", none)
        ffn_ms = gu_st["total_ms"] + dn_st["total_ms"]
        ffn_bytes = gu_st["bytes"] + dn_st["bytes"]
    elif timing and "gateup" not in stats:
        # one launch copies the misses and runs gate/up for all routed experts: it is
        # the dominant kernel and the host link bounds it
        cp, n_calls = stats["copy"], max(1, stats["router"]["launches"])
        avg_s = cp["total_ms"] / 1e3 / n_calls
        per_launch_bytes = cp["bytes"] / n_calls
        achieved = per_launch_bytes / avg_s / 1e9
        tname = {"a3b_decode": "copy_gateup_a3b_q8", "q4_decode": "copy_gateup_q4"}.get(wl.name)
        traffic = measured_traffic(args, tname, wl, budget) if tname and args.rho is None else None
        result["roofline"] = {"bound": "pcie", "kernel": "copy_gateup_kernel<8>" if wl.qtype == "q8_0"
                              else "copy_gateup_kernel<2>", "achieved": achieved,
                              "peak": PCIE_PEAK_GBS, "unit": "GB/s", "frac": achieved / PCIE_PEAK_GBS,
                              "traffic": traffic, "bytes_per_launch": per_launch_bytes,
                              "avg_launch_us": avg_s * 1e6,
                              "traffic_note": "FETCH_SIZE + WRITE_SIZE per launch: the misses' host "
                                              "reads and slot writes plus the hits' gate/up reads"}
        ffn_ms = stats["down"]["total_ms"]
        ffn_bytes = stats["down"]["bytes"]
    elif timing and wl.formats[0] in ("q4_k", "q6_k"):
        # K-quant decode: the misses' copies (copy kernel from the device work list) are the
        # dominant kernel, bound by the host link; gate/up and down run after them
        cp, n_calls = stats["copy"], max(1, stats["router"]["launches"])
        avg_s = cp["total_ms"] / 1e3 / n_calls
        per_launch_bytes = cp["bytes"] / n_calls
        achieved = per_launch_bytes / avg_s / 1e9
        traffic = measured_traffic(args, "copy_list_q4km", wl, budget) \
            if wl.name == "q4km_decode" and args.rho is None else None
        result["roofline"] = {"bound": "pcie", "kernel": "materialize_list_kernel", "achieved": achieved,
                              "peak": PCIE_PEAK_GBS, "unit": "GB/s", "frac": achieved / PCIE_PEAK_GBS,
                              "traffic": traffic, "bytes_per_launch": per_launch_bytes,
                              "avg_launch_us": avg_s * 1e6,
                              "traffic_note": "FETCH_SIZE + WRITE_SIZE per launch: the misses' host reads "
                                              "and slot writes"}
        ffn_ms = stats["gateup"]["total_ms"] + stats["down"]["total_ms"]
        ffn_bytes = stats["gateup"]["bytes"] + stats["down"]["bytes"]
    elif timing:
        gu = stats["gateup"]
        per_launch_bytes = gu["bytes"] / max(1, gu["launches"])
        avg_s = gu["total_ms"] / 1e3 / max(1, gu["launches"])
        achieved = per_launch_bytes / avg_s / 1e9
        traffic = measured_traffic(args, "gateup_a3b_q8", wl, budget) \
            if wl.qtype == "q8_0" and args.rho is None else None
        result["roofline"] = {"bound": "hbm", "kernel": "gateup_kernel<8>" if wl.qtype == "q8_0"
                              else "gateup_kernel<2>", "achieved": achieved, "peak": HBM_PEAK_GBS,
                              "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                              "bytes_per_launch": per_launch_bytes, "avg_launch_us": avg_s * 1e6}
        ffn_ms = stats["gateup"]["total_ms"] + stats["down"]["total_ms"]
        ffn_bytes = stats["gateup"]["bytes"] + stats["down"]["bytes"]
    result["extra"] = {
        "hit_rate": hits / max(1, hits + misses),
        "misses_per_token_layer": misses / (tokens * wl.n_layers),
        "materialized_bytes_per_token": mbytes / tokens,
        "evictions_per_step": evictions / args.steps,
        "us_per_layer_call": 1e6 * dt / (tokens * wl.n_layers),
        "h2d_peak_gb_per_s": h2d_peak,
        "h2d_1gib_gb_per_s": h2d_big,
        "static_plan": dict(plan, cache_percent=wl.cache_percent, target="HBM 288 GB"),
    }
    if timing and prefill and "copy" not in stats:
        fl = gu_st["flops"] + dn_st["flops"]
        result["extra"].update({
            "expert_ffn_tflops": fl / (ffn_ms * 1e9),
            "expert_ffn_frac_of_bf16_peak": fl / (ffn_ms * 1e9) / BF16_PEAK_TFLOPS,
            "down_tflops": dn_st["flops"] / (dn_st["total_ms"] * 1e9),
            "expert_ffn_note": "warm cache, no copies: the grouped GEMMs alone; algorithmic flops "
                               "(each GEMM also multiplies the lo activation term: 2x the MFMA work)",
            "kernels": stats,
        })
    if timing and "copy" in stats:
        cp = stats["copy"]
        if prefill:
            fl = gu_st["flops"] + dn_st["flops"]
            result["extra"]["expert_ffn_tflops"] = fl / (ffn_ms * 1e9)
            result["extra"]["expert_ffn_frac_of_bf16_peak"] = fl / (ffn_ms * 1e9) / BF16_PEAK_TFLOPS
            result["extra"]["expert_ffn_note"] = (
                "algorithmic flops (each GEMM also multiplies the lo activation term: 2x the MFMA "
                "work) over the GEMM launches' durations, which overlap the host copy kernel; "
                "running beside it slows them 2-4x")
        elif verify:
            result["extra"]["expert_ffn_note"] = (
                "int8-digit GEMVs, bytes over launch durations: the union down GEMVs of every "
                "window and, for windows whose union exceeds the slots, the union gate/up and down "
                "GEMVs per chunk, which overlap the host copy kernel")
        result["extra"].update({
            "expert_ffn_gb_per_s": ffn_bytes / (ffn_ms * 1e6),
            "expert_ffn_frac_of_hbm_peak": ffn_bytes / (ffn_ms * 1e6) / HBM_PEAK_GBS,
            "expert_ffn_kernels": ("union down GEMVs (their gate/up runs inside the copy launch) "
                                   "and the per-chunk union GEMVs of windows that take the "
                                   "host-table path")
                                  if verify and args.copy_mode == "kernel" else
                                  "gate/up + down" if "gateup" in stats else
                                  "down (gate/up runs inside the copy launch)",
            "copy_gb_per_s": cp["gb_per_s"],
            "copy_frac_of_best_measured_h2d": (cp["gb_per_s"] or 0) / max(h2d_peak, h2d_big or 0),
            "kernels": stats,
        })
    if not prefill and not verify:
        # the decode GEMVs read 13-27 MB per launch, where a launch's ramp is a large part
        # of its duration: the rocprofv3 kernel-trace durations of the down GEMV, a plain
        # read of its bytes in one launch and an empty launch (one clock for all three),
        # from profiles/decode_hbm_reference.json when it was taken on the current kernels
        path = os.path.join(args.profiles, "decode_hbm_reference.json")
        if os.path.exists(path):
            ref = json.load(open(path))
            if ref.get("kernel_sources_sha256_16") == kernel_sources_sha256_16() and wl.name in ref:
                result["extra"]["hbm_launch_reference"] = dict(ref[wl.name], clock=ref["clock"])
        st = stats.get("down") if timing else None
        if args.hbm_probe and st and st["launches"]:
            per = int(st["bytes"] // st["launches"]) // 16 * 16
            read_us, empty_us = probe_hbm_read(per, 50)
            log(f"HBM probe: {per} B per launch, plain read {read_us:.2f} us, "
                f"empty launch {empty_us:.2f} us (event clock)")
    if not prefill and not args.no_policy_bound:
        # the same run once more, untimed, keeping the slot trace: the routed sets of every
        # layer call, replayed through the offline miss bound (Belady's MIN) per layer
        tcache = MoeCache(wl.n_layers, wl.n_experts, wl.top_k, wl.hidden, wl.inter, wl.qtype,
                          hb.ptr, wl.store_bytes, budget, stream=torch.cuda.current_stream(),
                          residual=True, prenorm=True, trace=True, copy_mode=args.copy_mode,
                          score_evict=args.policy == "score")
        step(tcache)
        recs = tcache.read_trace()
        pol_misses = tcache.counters().misses
        tcache.close()
        sets = {}
        for layer, stp, e, _, _, _ in recs:
            sets.setdefault(layer, {}).setdefault(stp, []).append(e)
        bound = None
        if all(len(v) <= budget for per in sets.values() for v in per.values()):
            bound = sum(min_misses([per[k] for k in sorted(per)], wl.n_experts, budget)
                        for per in sets.values())
        result["extra"]["policy_bound"] = {
            "policy": args.policy,
            "policy_misses": pol_misses,
            "min_misses": bound,
            "policy_materialized_bytes_per_token": pol_misses * wl.payload_bytes / wl.n_tokens,
            "min_materialized_bytes_per_token": None if bound is None else
            bound * wl.payload_bytes / wl.n_tokens,
            "policy_over_min": None if not bound else pol_misses / bound,
            "what": "Belady MIN over the recorded routed sets of one run, per layer: no slot "
                    "policy can miss less on these routes"}
        log(f"offline bound: {args.policy} {pol_misses} misses, MIN {bound}")
    if verify:
        n_steps = len(windows)
        acc_drafts = sum(a for _, a, _ in windows)
        calls = n_steps * wl.n_layers
        result["extra"]["verify"] = {
            "horizon": wl.horizon, "accept_q": wl.accept_q, "steps": n_steps,
            "drafted": n_steps * wl.horizon, "accepted": acc_drafts,
            "accepted_frac": acc_drafts / max(1, n_steps * wl.horizon),
            "verified_tokens": n_steps * W,
            "mean_union_experts_per_layer_call": (hits + misses) / args.steps / calls,
            "materialized_bytes_per_generated_token": mbytes / tokens,
        }
        # the same tokens decoded one at a time on the same budget, cold
        cache.close()
        cache = MoeCache(wl.n_layers, wl.n_experts, wl.top_k, wl.hidden, wl.inter, wl.qtype, hb.ptr,
                         wl.store_bytes, budget, stream=torch.cuda.current_stream(), residual=True,
                         prenorm=True)
        h1 = torch.empty(wl.hidden, dtype=torch.float32, device="cuda")
        y1 = torch.empty_like(h1)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        for t in range(wl.n_tokens):
            h1.copy_(Xd[t])
            for l in range(wl.n_layers):
                cache.layer_forward(h1, Rd[l], l, y1, n_tokens=1)
                h1, y1 = y1, h1
        torch.cuda.synchronize()
        d1 = time.perf_counter() - t1
        c1 = cache.counters()
        result["extra"]["batch1_same_budget"] = {
            "tokens_per_s": wl.n_tokens / d1, "hit_rate": c1.hits / max(1, c1.hits + c1.misses),
            "materialized_bytes_per_token": c1.materialized_bytes / wl.n_tokens,
            "mean_experts_per_layer_call": (c1.hits + c1.misses) / (wl.n_tokens * wl.n_layers)}
        log(f"batch-1 decode on the same budget: {wl.n_tokens / d1:.1f} tok/s")
    cache.close()
    if args.calibrate_copy:
        a = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
        b = torch.empty_like(a)
        a.fill_(1)
        for _ in range(4):
            b.copy_(a)
        torch.cuda.synchronize()
        del a, b

    if not args.no_cpu_baseline:
        from threadpoolctl import threadpool_info
        from oracle.layer import run_stack
        n = args.cpu_sample_tokens
        log(f"cpu baseline: oracle on the first {n} tokens through all {wl.n_layers} layers")
        tc = time.perf_counter()
        if prefill or verify:  # a bounded sample: n tokens as one multi-token call per layer
            run_stack(X[:n], R, hb.array, wl, budget, decode=False, bf16=True, prenorm=True)
        else:
            run_stack(X[:n], R, hb.array, wl, budget, prenorm=True)
        cdt = time.perf_counter() - tc
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
        result["cpu_baseline"] = {"value": n / cdt, "unit": "tokens/s", "cores": threads,
                                  "kind": "oracle",
                                  "sample": f"first {n} of {wl.n_tokens} tokens, all {wl.n_layers} "
                                            f"layers, same inputs, fp64 numpy ({cdt:.1f} s)"}
    hb.free()
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
