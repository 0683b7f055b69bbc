#!/usr/bin/env python3
"""Benchmark of the DuoGPT layer solver on one MI355X.

One step = the whole per-layer path on the device: activation sparsification
and H/G/a accumulation, damped inverse Cholesky, score terms and the blocked
column sweep with lazy updates, for one LLaMA-shaped linear layer with its
calibration tokens already resident in HBM.  Prints one JSON line.
"""

from __future__ import annotations

import argparse
import json
import os
import platform
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_FP32_TFLOPS = 157.3    # MI355X dense fp32 MFMA
# Large fp32 products of the sweep's Y form run as six bf16 products of exactly split
# operands where the library's dispatch finds that faster (not the factorisation's, nor a
# quantised layer's); their rates are priced against a sixth of the bf16 peak
PEAK_SPLIT_TFLOPS = PEAK_BF16_TFLOPS / 6
PEAK_HBM_GBS = 8000.0       # MI355X HBM3E

# Bytes from beyond L2 per gram_bf16_kernel launch on this workload, from rocprofv3
# --pmc FETCH_SIZE and WRITE_SIZE runs (profiles/gram_kernel_llama2_70b_down_proj_hbm_traffic.md),
# each scaled by what the same counter reads for a plain 1 GiB streaming kernel
# (FETCH_SIZE x2.0, WRITE_SIZE x1.0).  Valid only for the kernel source they
# were taken on: any change to that file makes the figure unknown (null).
GRAM_TRAFFIC = {
    "source": "paper_2506_20194_amd/csrc/hessian.hip",
    "sha256": "ae7ee796037946224f1a1d4a6ad2d0c57fc180efc5734554dd5fc04c8d3a6f2e",
    "workload": "llama2_70b_down_proj",
    "fetch_kib": 169687254.2, "fetch_scale": 2.0,
    "write_kib": 3501162.9, "write_scale": 1.0,
}


# HBM bytes per dsc_gemv_kernel launch on the LLaMA-2-70B down_proj decode
# workload (profiles/dsc_gemv_kernel_llama2_70b_down_proj_decode.md), same
# counters and calibration as above.
DECODE_TRAFFIC = {
    "source": "paper_2506_20194_amd/csrc/decode.hip",
    "sha256": "23dcd580fb35eeb921eee599a5fb3cca4c74a19a44be110ecb7bfce42f29acc9",
    "workload": "llama2_70b_down_proj",
    "fetch_kib": 55165.1, "fetch_scale": 2.0,
    "write_kib": 2048.0, "write_scale": 1.0,
}


def packed_bytes(duo, n, k, block=128):
    """Packed operands in duo_prune_layer's workspace (0: no product of this size is
    split; 12 k^2 and more: the score product is): its size less its other parts."""
    ws = duo.duo_workspace_size
    parts = (4 * max(n, k) * k, 4 * k, ws(duo.DUO_OP_SCORE_TERMS, 0, k, 0, 0), ws(duo.DUO_OP_SWEEP, n, k, 0, block))
    return ws(duo.DUO_OP_PRUNE_LAYER, n, k, 0, block) - sum((b + 255) // 256 * 256 for b in parts)


def gram_traffic(workload, t=None):
    import hashlib

    t = GRAM_TRAFFIC if t is None else t
    if t["sha256"] is None:
        return None
    try:
        with open(os.path.join(ROOT, t["source"]), "rb") as f:
            same = hashlib.sha256(f.read()).hexdigest() == t["sha256"]
    except OSError:
        same = False
    if not same or workload != t["workload"]:
        return None
    return 1024.0 * (t["fetch_kib"] * t["fetch_scale"] + t["write_kib"] * t["write_scale"])


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="llama2_70b_down_proj")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-probes", action="store_true", help="skip the measured-peak probes")
    ap.add_argument("--nm", type=int, default=0, metavar="N",
                    help="N:4 semi-structured mask (App. B 2:4 variant) instead of the unstructured p_w mask")
    ap.add_argument("--decode", action="store_true",
                    help="dual-sparse decode GEMV over compressed columns (LLaMA-2-70B down_proj shape)")
    ap.add_argument("--quant", type=int, default=0, metavar="BITS",
                    help="joint RTN quantisation of the kept weights (Table 4), one grid per row and 128 columns")
    ap.add_argument("--act-order", action="store_true",
                    help="process channels by decreasing Hessian diagonal (App. B); adds the gathers to the step")
    ap.add_argument("--form", choices=["auto", "d", "y"], default="auto",
                    help="residual form of the sweep (duo_prune_layer's residual_form); auto: the library's choice")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="only run a device-to-device copy of MIB MiB (calibrates HBM byte counters)")
    return ap.parse_args()


def copy_probe(mib):
    """A plain streaming kernel of known size (y = -x over MIB MiB of fp32):
    its FETCH_SIZE / WRITE_SIZE counters give the factor that turns those
    counters into HBM bytes."""
    import torch

    n = mib << 20
    src = torch.ones(n // 4, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    torch.neg(src, out=dst)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(3):
        torch.neg(src, out=dst)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / 3
    print(json.dumps({"copy_probe_bytes_read": n, "copy_probe_bytes_written": n, "ms_per_copy": ms,
                      "GBs": 2 * n / (ms * 1e-3) / 1e9}), flush=True)


def _blas_threads():
    try:
        from threadpoolctl import threadpool_info

        return max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:  # pragma: no cover
        return len(os.sched_getaffinity(0))


def cpu_baseline(W, X, c):
    """The float64 oracle, untuned, timed on the host.

    The tiny layer runs end to end (R.prune_layer), with the host's BLAS
    threads and again on one core.  Larger layers run a bounded sample, each
    stage scaled by its complexity: stage 1 (m k^2) on the first ms tokens at
    full k, x m/ms; the damped inverse Cholesky and score terms (k^3) on the
    trailing t x t window of that H, G, a, x (k/t)^3; the sweep (n k^2) on the
    first ns rows over that window, x (n/ns)(k/t)^2."""
    import numpy as np

    from oracle import duo_ref as R

    cores = _blas_threads()
    n, k, m = c["n"], c["k"], c["m"]
    info = {"cpu": platform.processor() or platform.machine(),
            "blas": str(np.__config__.CONFIG.get("Build Dependencies", {}).get("blas", {}).get("name", "?"))}
    Wn = W.float().cpu().numpy()
    if k <= 1024:
        Xn = X.float().cpu().numpy()
        t = time.perf_counter()
        R.prune_layer(Wn, Xn, c["p_x"], c["p_w"], damp=c["damp"], B=c["block"])
        full = time.perf_counter() - t
        try:
            from threadpoolctl import threadpool_limits

            with threadpool_limits(limits=1):
                t = time.perf_counter()
                R.prune_layer(Wn, Xn, c["p_x"], c["p_w"], damp=c["damp"], B=c["block"])
                one = time.perf_counter() - t
        except ImportError:  # pragma: no cover
            one = None
        return {"value": full, "unit": "s/layer", "cores": cores, "kind": "oracle",
                "sample": "whole layer (R.prune_layer end to end)", "single_core_s": one, **info}
    ms = min(m, 2048 if k > 16384 else 8192)
    # the window must be large enough that the k^3 stages run at their
    # asymptotic rate (at 4096 the inverse takes almost as long as at 11008)
    tw = min(k, 8192 if k > 16384 else 4096)
    ns = min(n, 256 if k > 16384 else 512)
    Xs = X[:ms].float().cpu().numpy()
    t = time.perf_counter()
    H, G, a = R.hessian_terms(Xs, c["p_x"])
    t1 = time.perf_counter() - t
    del Xs
    w = slice(k - tw, k)
    Hw, Gw, aw = H[w, w].copy(), G[w, w].copy(), a[w].copy()
    del H, G
    t = time.perf_counter()
    L, _ = R.inverse_cholesky(Hw, c["damp"])
    t2 = time.perf_counter() - t
    t = time.perf_counter()
    fac, D, _ = R.score_terms(Gw, L, aw)
    t3 = time.perf_counter() - t
    t = time.perf_counter()
    R.sweep_blocked(Wn[:ns, w], L, D, fac, c["p_w"], c["block"])
    t4 = time.perf_counter() - t
    f1, f23, f4 = m / ms, (k / tw) ** 3, (n / ns) * (k / tw) ** 2
    stage = {"hessian": t1 * f1, "chol_inv": t2 * f23, "score_terms": t3 * f23, "sweep": t4 * f4}
    return {
        "value": sum(stage.values()), "unit": "s/layer", "cores": cores, "kind": "oracle",
        "sample": f"stage 1 on {ms} of {m} tokens at full k={k} (x{f1:g}); inverse Cholesky and score terms on "
                  f"the trailing {tw}x{tw} window (x(k/t)^3 = {f23:.4g}); sweep on {ns} of {n} rows over that "
                  f"window (x(n/ns)(k/t)^2 = {f4:.4g}); measured {t1 + t2 + t3 + t4:.1f} s of CPU work",
        "stage_s": stage, **info,
    }


def measured_peaks():
    """Probes of what this GPU reaches with library code, for context beside
    the published peaks: a device-to-device copy of 4 GiB (HBM), and torch.mm
    (hipBLASLt / rocBLAS) at 8192^3 in bf16 and fp32."""
    import torch

    dev = torch.device("cuda:0")
    out = {}
    src = torch.empty(1 << 30, dtype=torch.float32, device=dev).fill_(1.0)
    dst = torch.empty_like(src)

    def timed(fn, reps):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps * 1e-3

    sec = timed(lambda: dst.copy_(src), 5)
    out["hbm_copy_GBs"] = 2 * src.numel() * 4 / sec / 1e9
    del src, dst
    for dt, key in ((torch.bfloat16, "bf16_gemm_TFLOPs"), (torch.float32, "fp32_gemm_TFLOPs")):
        a = torch.randn((8192, 8192), device=dev).to(dt)
        b = torch.randn((8192, 8192), device=dev).to(dt)
        sec = timed(lambda: torch.mm(a, b), 10)
        out[key] = 2 * 8192 ** 3 / sec / 1e12
        del a, b
    out["note"] = "device copy of 4 GiB (read + write bytes) and torch.mm at 8192^3; library code, context only"
    return out


def bench_decode(args):
    """Dual-sparse decode: one GEMV per token over a pruned layer's compressed
    columns (only the channels whose activation survives are read).  The
    layer is the LLaMA-2-70B down_proj shape with a uniform random mask at the
    workload's weight sparsity standing in for a calibrated one."""
    import torch

    from paper_2506_20194_amd import duo
    from workloads import synth

    name = "llama2_70b_down_proj"
    c = synth.CONFIGS[name]
    n, k, p_x, p_w = c["n"], c["k"], c["p_x"], c["p_w"]
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(7)
    keep = torch.rand((n, k), generator=g, device=dev) >= p_w
    W = torch.where(keep, (0.02 * torch.randn((n, k), generator=g, device=dev)).to(torch.bfloat16),
                    torch.zeros((), dtype=torch.bfloat16, device=dev))
    words = (k + 31) // 32
    kp = torch.zeros((n, words * 32), dtype=torch.int64, device=dev)
    kp[:, :k] = keep.to(torch.int64)
    mask = (kp.view(n, words, 32) << torch.arange(32, device=dev)).sum(-1).to(torch.int32)
    del kp
    comp = duo.dsc_compress(W, mask)
    ws = duo.dsc_workspace(n, k, dev)
    y = torch.empty(n, dtype=torch.float32, device=dev)
    T = max(16, args.steps * 16)
    xs = (torch.randn((T, k), generator=g, device=dev) * torch.exp(torch.randn((T, k), generator=g, device=dev))
          ).to(torch.bfloat16)
    # bytes each token's GEMV must fetch: the active channels' mask words,
    # chunk offsets and kept values, plus x and y
    xh = duo.duo_act_sparsify(xs, p_x)
    act = xh != 0
    cnt = (comp["col_ptr"][1:] - comp["col_ptr"][:-1]).to(torch.float64)
    per_col = 4 * ((n + 31) // 32) + 2 * ((n + 255) // 256)
    fetched = (act.to(torch.float64) * (per_col + 2 * cnt)).sum(1) + 2 * k + 4 * n
    for t in range(min(T, 4)):
        duo.dsc_gemv(comp, xs[t], p_x, ws=ws, out=y)
    # cold caches, as in a decode step (every other layer runs between two
    # uses of this one): a 1 GiB buffer, four times the last-level cache, is
    # read before each token; each call is timed on its own
    flush = torch.zeros(1 << 28, dtype=torch.float32, device=dev)
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(T)]

    def timed(fn):
        for t in range(T):
            flush.sum()
            evs[t][0].record()
            fn(t)
            evs[t][1].record()
        torch.cuda.synchronize()
        return sum(a.elapsed_time(b) for a, b in evs) * 1e3 / T

    torch.cuda.synchronize()
    us_call = timed(lambda t: duo.dsc_gemv(comp, xs[t], p_x, ws=ws, out=y))
    # the GEMV kernel alone, in a second pass (its events would sit between
    # the call's kernels in the first)
    duo.duo_profile_enable(True)
    duo.duo_profile_read("decode")
    timed(lambda t: duo.dsc_gemv(comp, xs[t], p_x, ws=ws, out=y))
    dec_ms, dec_n = duo.duo_profile_read("decode")
    duo.duo_profile_enable(False)
    us_kernel = dec_ms * 1e3 / max(dec_n, 1)
    gbs = float(fetched.mean()) / (us_kernel * 1e-6) / 1e9
    # dense bf16 GEMV on the same layer for context, under the same flushes
    for _ in range(3):
        torch.mm(W, xs[0].view(k, 1))
    dense_us = timed(lambda t: torch.mm(W, xs[t].view(k, 1)))
    line = {
        "metric": "us per dual-sparse decode GEMV (one token, compressed columns)",
        "value": us_call, "unit": "us/token", "n_gpus": 1, "steps": T, "warmup": 4, "ms_per_step": us_call / 1e3,
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "bf16 weights, fp32 accumulate",
        "data": "synthetic (uniform random mask at the workload's weight sparsity); caches flushed before each token",
        "config": {"workload": name + " decode", "n": n, "k": k, "p_x": p_x, "p_w": p_w,
                   "nnz": int(comp["col_ptr"][k].item()), "parallelism": "single GPU"},
        "roofline": {"bound": "hbm", "kernel": "dsc_gemv_kernel", "achieved": gbs, "peak": PEAK_HBM_GBS,
                     "unit": "GB/s", "frac": gbs / PEAK_HBM_GBS, "traffic": gram_traffic(name, DECODE_TRAFFIC),
                     "us_per_launch": us_kernel,
                     "bytes_per_launch": float(fetched.mean())},
        "dense_bf16_gemv_us": dense_us,
    }
    print(json.dumps(line))


def bench_block(args):
    """The LLaMA-2-7B decoder block pruned group by group (7 linears, 4 shared
    Hessians) on 128 x 2048 tokens; the forward passes of the two activation
    streams between groups are reported separately from the solver."""
    import torch

    from paper_2506_20194_amd import block
    from workloads import synth

    name = args.workload
    c = synth.BLOCKS[name]
    cfg = synth.block_cfg(name)
    dev = torch.device("cuda:0")
    h, w = synth.block_inputs(name, device=dev)
    runs = []
    for i in range(args.warmup + args.steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = block.prune_block(h, w, cfg, c["p_x"], c["p_w"], damp=c["damp"], block=c["block"], timing=True)
        wall = time.perf_counter() - t0
        if i >= args.warmup:
            runs.append((out["ms"], wall))
        del out
    ms = {k: sum(r[0][k] for r in runs) / len(runs) for k in runs[0][0]}
    solve_ms = sum(v for k, v in ms.items() if k.startswith("solve"))
    line = {
        "metric": "s/block for DuoGPT pruning of a LLaMA-2-7B-shaped decoder block (solver time; the two "
                  "activation streams' forward passes reported separately)",
        "value": solve_ms / 1e3, "unit": "s/block", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": solve_ms, "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16 MFMA (H, G) + fp32", "data": "synthetic",
        "config": {"workload": name, "d": c["d"], "ffn": c["ffn"], "heads": c["heads"], "head_dim": c["head_dim"],
                   "tokens": cfg["nseq"] * cfg["seq_len"], "p_x": c["p_x"], "p_w": c["p_w"], "block": c["block"],
                   "damp": c["damp"], "parallelism": "single GPU"},
        "group_solve_ms": {k: v for k, v in ms.items() if k.startswith("solve")},
        "forward_ms_both_streams": ms["forward"],
        "wall_s_per_block": sum(r[1] for r in runs) / len(runs),
    }
    print(json.dumps(line), flush=True)


def main():
    args = parse()
    if args.nm and (args.act_order or not 0 < args.nm <= 4):
        sys.exit("bench.py: --nm takes N in 1..4 and is not combined with --act-order")
    if args.quant and (args.act_order or not 2 <= args.quant <= 8):
        sys.exit("bench.py: --quant takes 2..8 bits and is timed without --act-order")
    if args.gpus != 1:
        print(f"bench.py: the solver runs on one GPU only (asked for --gpus {args.gpus}); "
              "the multi-GPU path is a design note, not implemented", file=sys.stderr)
        sys.exit(2)
    if args.copy_probe:
        copy_probe(args.copy_probe)
        return
    from workloads import synth as _synth

    if args.decode:
        bench_decode(args)
        return
    if args.workload in _synth.BLOCKS:
        bench_block(args)
        return
    import torch

    from paper_2506_20194_amd import duo
    from workloads import synth

    c = synth.CONFIGS[args.workload]
    n, k, m, B = c["n"], c["k"], c["m"], c["block"]
    dev = torch.device("cuda:0")
    W, X = synth.config_inputs(args.workload, device=dev)
    H = torch.zeros((k, k), dtype=torch.float32, device=dev)
    G = torch.zeros((k, k), dtype=torch.float32, device=dev)
    a = torch.zeros(k, dtype=torch.float32, device=dev)
    ws_h = duo.workspace(duo.DUO_OP_HESSIAN, 0, k, m, 0, dev)
    ws_c = duo.workspace(duo.DUO_OP_CHOL_INV, 0, k, 0, 0, dev)
    ws_p = duo.workspace(duo.DUO_OP_PRUNE_LAYER, n, k, 0, B, dev)
    W_out = torch.empty((n, k), dtype=torch.float32, device=dev)
    lowp = torch.empty((n, k), dtype=W.dtype, device=dev)
    mask = torch.empty((n, (k + 31) // 32), dtype=torch.int32, device=dev)

    if args.act_order:
        hdiag = torch.zeros(k, dtype=torch.float64, device=dev)
        Hp, Gp = torch.empty_like(H), torch.empty_like(G)
        ap_, Wp = torch.empty((1, k), dtype=torch.float32, device=dev), torch.empty_like(W)
        W_out_p, lowp_p, mask_p = torch.empty_like(W_out), torch.empty_like(lowp), torch.empty_like(mask)

    def step(check=False):
        H.zero_()
        G.zero_()
        a.zero_()
        if not args.act_order:
            duo.duo_hessian_accum(X, H, c["p_x"], G=G, a=a, ws=ws_h)
            info = duo.duo_chol_inv(H, c["damp"], ws=ws_c, sync=check)
            duo.duo_prune_layer(W, H, G, a, c["p_w"], B, ws=ws_p, out=(W_out, lowp, mask, None), nm_n=args.nm,
                                quant=(args.quant, 128) if args.quant else None, form=args.form)
            return info
        hdiag.zero_()
        duo.duo_hessian_accum(X, H, c["p_x"], G=G, a=a, ws=ws_h, hdiag=hdiag)
        perm, inv = duo.duo_act_order(hdiag)
        duo.duo_permute(H, perm, perm, out=Hp)
        duo.duo_permute(G, perm, perm, out=Gp)
        duo.duo_permute(a.view(1, k), None, perm, out=ap_)
        duo.duo_permute(W, None, perm, out=Wp)
        info = duo.duo_chol_inv(Hp, c["damp"], ws=ws_c, sync=check)
        duo.duo_prune_layer(Wp, Hp, Gp, ap_.view(k), c["p_w"], B, ws=ws_p, out=(W_out_p, lowp_p, mask_p, None),
                            form=args.form)
        duo.duo_permute(W_out_p, None, inv, out=W_out)
        duo.duo_permute(lowp_p, None, inv, out=lowp)
        duo.duo_permute_mask(mask_p, k, inv, out=mask)
        return info

    lam, fail = step(check=True)  # also checks that the damped Hessian factors
    assert fail == -1
    for _ in range(max(0, args.warmup - 1)):
        step()
    torch.cuda.synchronize()
    # the timed steps carry no per-kernel events; a second, profiled pass of
    # the same steps gives the stage split and the Gram kernel's launch time
    # one event at every step boundary (markers on the stream, no kernel is
    # touched): the mean over the K steps is the reported time, the median of
    # the per-step times is reported beside it
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    ev[0].record()
    for i in range(args.steps):
        step()
        ev[i + 1].record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    ms_step = ev[0].elapsed_time(ev[-1]) / args.steps
    ms_step_median = float(statistics.median(ev[i].elapsed_time(ev[i + 1]) for i in range(args.steps)))
    duo.duo_profile_enable(True)
    for name in duo.PROF:
        duo.duo_profile_read(name)
    p0 = torch.cuda.Event(enable_timing=True)
    p1 = torch.cuda.Event(enable_timing=True)
    p0.record()
    for _ in range(args.steps):
        step()
    p1.record()
    torch.cuda.synchronize()
    duo.duo_profile_enable(False)
    ms_step_profiled = p0.elapsed_time(p1) / args.steps
    prof = {name: duo.duo_profile_read(name) for name in duo.PROF}

    # sanity: exact number of pruned weights
    kept = int(duo.unpack_mask(mask, k).sum().item())
    expect_pruned = n * k * args.nm // 4 if args.nm else int((c["p_w"] * n * k) + 0.5)
    assert n * k - kept == expect_pruned, (n * k - kept, expect_pruned)

    per = lambda name: prof[name][0] / max(prof[name][1], 1)     # ms per launch
    per_step = lambda name: prof[name][0] / args.steps              # ms per layer
    # Stage 1's algorithmic work: H on and above its diagonal, k(k+1)/2 dot
    # products over m tokens (2 flop per multiply-add), and the part of G the
    # solver reads, likewise its upper triangle (Eq. 7 uses Q = G L only on and
    # above its diagonal); all of G (2 k^2 m) with act_order, which permutes it
    g_flop = 2 * k * k * m if args.act_order else k * (k + 1) * m
    gram_flop_step = k * (k + 1) * m + g_flop
    gram_launches = prof["gram"][1] / args.steps
    gram_tflops = gram_flop_step / gram_launches / (per("gram") * 1e-3) / 1e12
    hess_flop = gram_flop_step
    hess_tflops = hess_flop / (per_step("hessian") * 1e-3) / 1e12
    sweep_bytes = 16 * n * k
    sweep_ms = per_step("select") + per_step("inblock")
    sweep_gbs = sweep_bytes / (sweep_ms * 1e-3) / 1e9
    # residual form of the sweep: the library's automatic choice (DUO_FORM_AUTO)
    # is the Y form (no D) from k = 6144 (with quantisation: groups of the block's width)
    yform = args.form == "y" or (args.form == "auto" and (not args.quant or B == 128) and k >= 6144)
    # lazy updates: the two terms (E L^T and W0 D, or (Y - E) L^T and W0 U) of
    # each block over the columns after it, 2 n k (k - B) flop; the Y form adds
    # the block-start products Y[:, blk] L[blk, blk]^T, 2 n B (k - B)
    trail_flop = 2 * n * k * (k - B) + (2 * n * B * (k - B) if yform else 0)
    trail_tflops = trail_flop / (per_step("trail") * 1e-3) / 1e12
    # A3 + A4 on the implemented route: UL factorisation k^3/3 + triangular
    # inverse k^3/3 + upper triangle of Q = G L k^3/3 (+ D = U L^T k^3/3 in the
    # D form); the survey's count (8/3) k^3 is for the plain route (explicit
    # inverse, Cholesky, full products) and is printed beside it
    chol_score_flop = (3 if yform else 4) * k ** 3 / 3
    chol_score_flop_plain = 8 * k ** 3 / 3
    split = packed_bytes(duo, n, k) if yform and not args.quant else 0
    f32_peak = PEAK_SPLIT_TFLOPS if split else PEAK_FP32_TFLOPS
    score_peak = PEAK_SPLIT_TFLOPS if split >= 12 * k * k else PEAK_FP32_TFLOPS
    # the factorisation's two thirds of k^3 at the fp32 peak, the score terms' rest at theirs
    chol_score_peak = chol_score_flop / (2 * k ** 3 / 3 / PEAK_FP32_TFLOPS + (chol_score_flop - 2 * k ** 3 / 3) / score_peak)
    # the Gram kernel multiplies in the calibration input's precision: bf16
    # MFMA for bf16 inputs, fp32 MFMA for fp32 inputs
    gram_peak = PEAK_BF16_TFLOPS if c["x_dtype"] == torch.bfloat16 else PEAK_FP32_TFLOPS
    line = {
        "metric": "s/layer for OBC prune of LLaMA-shaped linears; Hessian TFLOP/s; sweep GB/s",
        "value": ms_step / 1e3,
        "unit": "s/layer",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": ("bf16" if gram_peak == PEAK_BF16_TFLOPS else "fp32") + " MFMA (H, G) + fp32",
        "data": "synthetic",
        "config": {"workload": args.workload, "n": n, "k": k, "m": m, "p_x": c["p_x"], "p_w": c["p_w"],
                   "block": B, "damp": c["damp"], "x_dtype": str(c["x_dtype"]).replace("torch.", ""),
                   "inputs": c["kind"], "act_order": bool(args.act_order),
                   "mask": f"{args.nm}:4" if args.nm else "unstructured",
                   "quant": f"int{args.quant} g128" if args.quant else None,
                   "residual_form": "Y" if yform else "D", "parallelism": "single GPU"},
        "roofline": {"bound": "mfma", "kernel": f"gram_{'bf16' if gram_peak == PEAK_BF16_TFLOPS else 'f32'}_kernel (H, G)",
                     "achieved": gram_tflops, "peak": gram_peak, "unit": "TFLOP/s", "frac": gram_tflops / gram_peak,
                     "traffic": gram_traffic(args.workload), "ms_per_launch": per("gram"), "flop_per_launch": gram_flop_step / gram_launches},
        "hessian_tflops": hess_tflops,
        "hessian_frac": hess_tflops / gram_peak,
        "sweep_gbs": sweep_gbs,
        "sweep_frac": sweep_gbs / PEAK_HBM_GBS,
        "trailing_tflops": trail_tflops,
        "trailing_frac": trail_tflops / f32_peak,
        "chol_score_tflops": chol_score_flop / ((per_step("chol") + per_step("score")) * 1e-3) / 1e12,
        "chol_score_frac": chol_score_flop / ((per_step("chol") + per_step("score")) * 1e-3) / 1e12 / chol_score_peak,
        "fp32_product_peak_TFLOPs": f32_peak,
        "chol_score_flop_count": ("k^3 (implemented route, Y form: no D)" if yform else "(4/3) k^3 (implemented route)")
                                 + "; plain route (8/3) k^3 gives "
                                 f"{chol_score_flop_plain / ((per_step('chol') + per_step('score')) * 1e-3) / 1e12:.1f} TFLOP/s",
        "stage_ms": {name: per_step(name) for name in duo.PROF},
        "ms_per_step_median": ms_step_median,
        "ms_per_step_with_stage_events": ms_step_profiled,
        "wall_s_timed": wall,
        "lambda": lam,
    }
    del H, G, a, ws_h, ws_c, ws_p, W_out, lowp, mask
    torch.cuda.empty_cache()
    if not args.no_probes:
        pk = measured_peaks()
        pk["gram_frac_of_measured_bf16"] = gram_tflops / pk["bf16_gemm_TFLOPs"]
        pk["trailing_frac_of_measured_fp32"] = trail_tflops / pk["fp32_gemm_TFLOPs"]
        pk["sweep_frac_of_measured_copy"] = sweep_gbs / pk["hbm_copy_GBs"]
        line["measured_peaks"] = pk
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline(W, X, c)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
