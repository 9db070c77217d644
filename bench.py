#!/usr/bin/env python3
"""Benchmark of the OmniCache cached attention layer on one MI355X.

Workload: an SD3-1024-like joint-attention layer (64x64 = 4096 image tokens
plus 333 uncached text tokens, C=1536, 24 heads x 64, bf16) with Token Cache
at ratio r, seeded synthetic inputs (oc_synth), weights ~ N(0, 1/C).  One
"step" is one oc_layer_cached call on a new denoising-step input with a warm
layer cache: match, select, reduced attention, in-place restoration.

Prints one JSON line: throughput in layer tokens per second at r (default
0.5), latency and speed-up against the uncached layer at r = 0.25/0.5/0.75,
the roofline of the dominant kernel (live HIP-event stage timing), and the
CPU oracle timed on a bounded sample on this host.
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

METRIC = "cached attn-layer tokens/sec & latency vs uncached at r; MFMA % / HBM GB/s"
PEAK_MFMA_TFLOPS = 2516.6     # MI355X dense bf16 / fp16 MFMA
PEAK_HBM_GBS = 8000.0         # MI355X HBM3E
# Counter summaries of each workload's kernels (rocprofv3 FETCH_SIZE /
# WRITE_SIZE runs, scaled by a copy kernel of known size) and the sources each
# was taken on.
PROFILES = {
    "sd3_1024": os.path.join(ROOT, "profiles", "sd3_1024_r050_kernels.md"),
    "latte_spatial": os.path.join(ROOT, "profiles", "latte_spatial_frame_cache_kernels.md"),
    "latte_temporal": os.path.join(ROOT, "profiles", "latte_temporal_block_cache_kernels.md"),
    "svdxt_level": os.path.join(ROOT, "profiles", "svdxt_level_frame_token_cache_kernels.md"),
    "svdxt_level_k4": os.path.join(ROOT, "profiles", "svdxt_level_k4_frame_token_cache_kernels.md"),
    "sd3_ffn": os.path.join(ROOT, "profiles", "sd3_1024_ffn_r050_kernels.md"),
}
PROFILE = PROFILES["sd3_1024"]
_COMMON = ("oc_attn_common.h", "oc_device.h")
_TILES = ("oc_ring_tile.h", "oc_mfma_tile.h", "oc_gemm_epi.h")
KERNEL_SOURCES = {
    "flash": ("k_flash.hip", "k_flash_split.hip") + _COMMON,
    "proj_qkv": ("k_proj.hip",) + _TILES + _COMMON,
    "proj_out": ("k_proj.hip",) + _TILES + _COMMON,
    "match": ("k_match.hip", "oc_ring_tile.h", "oc_dma_tile.h", "oc_mfma_tile.h", "oc_groups.h", "oc_device.h"),
    "select": ("k_select.hip", "oc_groups.h", "oc_block.h", "oc_device.h"),
    "inv_norm": ("k_match.hip", "oc_device.h"),
    "frame_gram": ("k_frame.hip", "oc_device.h"),
    "frame_final": ("k_frame.hip", "oc_device.h"),
    "attn_short": ("k_flash.hip",) + _COMMON,
    "qkv_attn_short": ("k_short.hip",) + _TILES + _COMMON,
    "compact": ("k_compact.hip", "oc_groups.h", "oc_device.h"),
    "ffn_up": ("k_ffn.hip",) + _TILES + _COMMON,
    "ffn_down": ("k_ffn.hip",) + _TILES + _COMMON,
}


def kernel_source_hash(stage):
    """First 16 hex digits of the SHA-1 of the stage's kernel sources."""
    import hashlib
    h = hashlib.sha1()
    for f in KERNEL_SOURCES[stage]:
        with open(os.path.join(ROOT, "paper_2607_23844_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def kernel_traffic(stage, workload="sd3_1024"):
    """HBM bytes per launch of a stage's kernel from the workload's committed
    counter summary, or None when there is none or its sources changed since."""
    try:
        with open(PROFILES[workload]) as fh:
            kv = dict((k.strip(), v.strip()) for k, v in
                      (l.split(":", 1) for l in fh.read().splitlines() if l.startswith(("traffic.", "sha1."))))
        if stage not in KERNEL_SOURCES or kv[f"sha1.{stage}"] != kernel_source_hash(stage):
            return None
        return int(float(kv[f"traffic.{stage}"]))
    except (OSError, KeyError, ValueError):
        return None


def stage_work(shape, cfg, pl, n_ctx=0):
    """Algorithmic work per launch of each stage of one layer call:
    {stage: (flop, bytes)}, what the method itself must compute and move
    (bf16 operands, 2 bytes; fp32 norms).  Selection, compaction and the
    frame-stage reductions are latency-bound and have no entry."""
    C, hd = shape.C, shape.heads * shape.head_dim
    FN = shape.F * shape.N
    rows = pl.n_kept + n_ctx
    lk = pl.seq_len + (n_ctx if pl.n_seq == 1 else 0)
    attn_flop = 4.0 * pl.n_seq * lk * lk * hd
    # candidates that exist: groups of a frame pair hold all tokens of two
    # frame-patches but one's representatives, the others of one (n_src_max is
    # the larger of the two)
    n_cand, D = pl.n_groups * pl.n_src_max, pl.n_dst_max
    if cfg.gran == "frame_token":
        n = FN // shape.F
        n_cand = (shape.F - 2 * pl.n_frame_cached) * (n - n // 4) + pl.n_frame_cached * (2 * n - n // 4)
    K = shape.F * C if cfg.gran == "block" else C
    frames = cfg.gran in ("frame", "frame_token")
    return {
        "proj_qkv": (2.0 * rows * C * 3 * hd, 2.0 * (rows * C + 3 * hd * C + 3 * rows * hd)),
        "flash": (attn_flop, 2.0 * 4 * rows * hd),
        "attn_short": (attn_flop, 2.0 * 4 * rows * hd),
        "qkv_attn_short": (2.0 * rows * C * 3 * hd + attn_flop, 2.0 * (rows * C + 3 * hd * C + rows * hd)),
        "proj_out": (2.0 * rows * hd * C, 2.0 * (rows * hd + hd * C + rows * C)),
        "match": (2.0 * n_cand * D * K, 2.0 * FN * C + 4.0 * FN),
        "inv_norm": (2.0 * FN * C, 2.0 * FN * C + 4.0 * FN),
        "frame_gram": (2.0 * shape.F * shape.F * shape.N * C if frames else 0.0,
                       2.0 * FN * C + (4.0 * FN if cfg.gran == "frame_token" else 0.0)),
        "gather": (0.0, 2.0 * pl.n_kept * C * 2.0),
        "restore": (0.0, 2.0 * pl.n_kept * C * 2.0),
        "residual": (float(FN * C), 3.0 * FN * C * 2.0),
    }


def roofline_of(flop, nbytes, avg_us):
    """Bound (the resource whose ideal time is longer), achieved rate and
    fraction of MI355X peak for one launch of avg_us."""
    t_mfma = flop / (PEAK_MFMA_TFLOPS * 1e12)
    t_hbm = nbytes / (PEAK_HBM_GBS * 1e9)
    sec = avg_us * 1e-6
    if t_mfma >= t_hbm and flop > 0:
        ach = flop / sec / 1e12
        return dict(bound="mfma", achieved=round(ach, 2), peak=PEAK_MFMA_TFLOPS, unit="TFLOP/s",
                    frac=round(ach / PEAK_MFMA_TFLOPS, 4))
    ach = nbytes / sec / 1e9
    return dict(bound="hbm", achieved=round(ach, 1), peak=PEAK_HBM_GBS, unit="GB/s", frac=round(ach / PEAK_HBM_GBS, 4))


def kernel_table(stages, K, work, workload):
    """Per-stage live timing (HIP events stamped at each kernel's start and
    end) with its roofline where the stage has algorithmic work, and the
    roofline object of the dominant stage (largest time).  A stage may run
    several kernels per call (split-K similarity and its reduction, the two
    compaction passes): avg_us is the mean kernel launch, us_per_step the
    stage's time per call, which the roofline and traffic figures use."""
    kernels = {}
    for name, (tot_ms, n) in stages.items():
        avg_us = tot_ms * 1e3 / max(n, 1)
        step_us = tot_ms * 1e3 / K
        d = dict(avg_us=round(avg_us, 3), launches_per_step=round(n / K, 3), us_per_step=round(step_us, 3))
        tr = kernel_traffic(name, workload)
        if tr is not None:
            d["traffic"] = tr
        if name in work and (work[name][0] > 0 or work[name][1] > 0):
            d.update(roofline_of(work[name][0], work[name][1], step_us))
        kernels[name] = d
    dom = max(stages, key=lambda s: stages[s][0])
    roof = None
    if dom in work:
        step_us = stages[dom][0] * 1e3 / K
        flop, nbytes = work[dom]
        r = roofline_of(flop, nbytes, step_us)
        roof = dict(kernel=dom, **r, traffic=kernel_traffic(dom, workload), avg_us=round(step_us, 3),
                    launches_per_step=round(stages[dom][1] / K, 3),
                    algorithmic_per_launch=flop if r["bound"] == "mfma" else nbytes)
    return kernels, roof


def stage_times(fn, inputs, K):
    """{stage: (total ms, launches)} over K calls, with the stage timer attached."""
    import torch
    import paper_2607_23844_amd as oc
    timer = oc.StageTimer()
    with timer:
        for i in range(K):
            fn(inputs[i % len(inputs)])
    torch.cuda.synchronize()
    return timer.collect()


def step_percentiles(fn, inputs, K):
    """Per-step latency (µs) from events between consecutive steps: p10, p50, p90."""
    import numpy as np
    import torch
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(K + 1)]
    ev[0].record()
    for i in range(K):
        fn(inputs[i % len(inputs)])
        ev[i + 1].record()
    torch.cuda.synchronize()
    d = np.array([ev[i].elapsed_time(ev[i + 1]) * 1e3 for i in range(K)])
    return dict(p10_us=round(float(np.percentile(d, 10)), 2), p50_us=round(float(np.percentile(d, 50)), 2),
                p90_us=round(float(np.percentile(d, 90)), 2))


def graph_latency(run, x, K, pairs=4):
    """A warm step captured once in a HIP graph, against the same step
    launched eagerly: {graph_us, eager_us}, medians over `pairs` interleaved
    blocks of K replays and K eager calls (the clock settles over the first
    blocks, so the two are compared in the same phase of the run)."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run.use_current_stream()
        for _ in range(3):
            run(x)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run.use_current_stream()
        run(x)
    run.use_current_stream()
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()

    def block(fn):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(K):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / K

    gs, es = [], []
    for _ in range(pairs):
        es.append(block(lambda: run(x)))
        gs.append(block(g.replay))
    gs.sort()
    es.sort()
    return dict(graph_us=round(gs[len(gs) // 2], 2), eager_us=round(es[len(es) // 2], 2))


def timed_ms(fn, inputs, K, W):
    import torch
    for i in range(W):
        fn(inputs[i % len(inputs)])
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(K):
        fn(inputs[i % len(inputs)])
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / K


def _bf16_dev(a, dev):
    import numpy as np
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(dev)


def run_other_configs(args):
    """The Latte-like spatial (Frame Cache) and temporal (Block Cache) layers
    and the SVD-XT-like level (Frame+Token spatial layer with whole-frame or
    patch-local token matching, uncached temporal layer): warm cached latency
    against the uncached layer, each kernel's live time, and the roofline of
    the layer's dominant kernel."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import FullRunner, LayerRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    K, Wm = args.cfg_steps, 3
    out = {}
    # SVD-XT twice: token matching over whole frames (k = 1) and patch-local
    # (k = 4: 4x4 patches, the paper's hierarchy for lower matching cost)
    for key, name in (("latte_spatial_frame_cache", "latte_spatial"), ("latte_temporal_block_cache", "latte_temporal"),
                      ("svdxt_level_frame_token_cache", "svdxt_level"),
                      ("svdxt_level_frame_token_cache_k4", "svdxt_level_k4")):
        if args.only and args.only != name:
            continue
        wl = make_workload(name, 3)
        xs = [_bf16_dev(s, dev) for s in wl.steps]
        W = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
        shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, 0, "bf16")
        cfg = oc.Cfg(wl.gran, r=wl.r, r_frame=wl.r_frame, patch_k=wl.patch_k)
        full = FullRunner(shape, oc.Cfg(wl.gran, 0.0, 0.0, 1), W, dev)
        full_ms = timed_ms(full, xs, K, Wm)
        # the uncached layer's stages, live time per call (µs)
        ust = stage_times(full, xs, K)
        uncached_stages = {st: round(t * 1e3 / K, 3) for st, (t, n) in ust.items()}
        run = LayerRunner(shape, cfg, W, dev)
        run(xs[0])
        ms = timed_ms(run, xs[1:], K, Wm)
        stages = stage_times(run, xs[1:], K)
        pl = oc.plan(shape, cfg)
        kernels, roof = kernel_table(stages, K, stage_work(shape, cfg, pl), name)
        tokens = wl.F * wl.H * wl.W
        d = dict(workload=f"F={wl.F}, {wl.H}x{wl.W} tokens, C={wl.C}, {wl.heads}x{wl.head_dim}, bf16, {wl.gran} "
                          f"r={wl.r} r_frame={wl.r_frame} patch_k={wl.patch_k}",
                 cached_us=round(ms * 1e3, 2), uncached_us=round(full_ms * 1e3, 2),
                 speedup_vs_uncached=round(full_ms / ms, 4), tokens_per_s=round(tokens / (ms * 1e-3), 1),
                 retained_tokens=pl.n_kept, sequences=f"{pl.n_seq}x{pl.seq_len}", roofline=roof, kernels=kernels,
                 uncached_stages_us=uncached_stages)
        if wl.t_weights is not None:
            TW = {k: _bf16_dev(v, dev) for k, v in wl.t_weights.items()}
            temporal = FullRunner(shape, oc.Cfg("block", 0.0, 0.0, 1), TW, dev)
            t_ms = timed_ms(temporal, xs, K, Wm)
            d.update(temporal_layer_us=round(t_ms * 1e3, 2),
                     level_cached_us=round((ms + t_ms) * 1e3, 2), level_uncached_us=round((full_ms + t_ms) * 1e3, 2),
                     level_speedup=round((full_ms + t_ms) / (ms + t_ms), 4))
            del temporal, TW
        out[key] = d
        del run, full, xs, W
        torch.cuda.empty_cache()
    return out


def run_ffn(args):
    """The feed-forward sublayer of the SD3-like block under the attention's
    selection at r = 0.5 (2048 of 4096 image tokens, hidden 4C = 6144): the
    cached FFN (retained rows only, written in place) against the uncached
    one (every token), each kernel's live time and roofline."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import FfnRunner, LayerRunner
    from oc_synth import ffn_weights, make_workload

    dev = torch.device("cuda:0")
    K, Wm = args.cfg_steps, 3
    wl = make_workload("sd3_1024", 2)
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, wl.n_ctx, "bf16")
    cfg = oc.Cfg("token", r=0.5)
    xs = [_bf16_dev(s, dev) for s in wl.steps]
    W = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
    ctx = _bf16_dev(wl.ctx, dev)
    hidden = 4 * wl.C
    Wf = {k: _bf16_dev(v, dev) for k, v in ffn_weights(wl.C, hidden, "bf16").items()}
    attn = LayerRunner(shape, cfg, W, dev, ctx)
    attn(xs[0])
    _, _, tr = oc.layer_cached(xs[1], W, attn.cache, shape, cfg, ctx=ctx, ws=attn.ws, trace=True)
    kept = tr["kept_idx"].clone()
    cached = FfnRunner(shape, Wf, kept, dev)
    full = FfnRunner(shape, Wf, None, dev)
    ms = timed_ms(cached, xs, K, Wm)
    full_ms = timed_ms(full, xs, K, Wm)
    stages = stage_times(cached, xs, K)
    n, C = kept.numel(), wl.C
    work = {"ffn_up": (2.0 * n * C * hidden, 2.0 * (n * C + hidden * C + n * hidden)),
            "ffn_down": (2.0 * n * hidden * C, 2.0 * (n * hidden + C * hidden + n * C))}
    kernels, roof = kernel_table(stages, K, work, "sd3_ffn")
    return dict(workload=f"SD3-1024-like FFN: 4096 image tokens, C={C}, hidden {hidden}, GELU (tanh), bf16, the "
                         f"attention's r=0.5 selection ({n} retained rows)",
                cached_us=round(ms * 1e3, 2), uncached_us=round(full_ms * 1e3, 2),
                speedup_vs_uncached=round(full_ms / ms, 4), retained_rows=n, roofline=roof, kernels=kernels)


def run_blocks(args):
    """Spatial + temporal blocks with all three caches at the paper's
    operating points (Latte r_f/r_b/r_t = 30/40/20, SVD-XT 50/40/50, the
    latter with patch-local 4x4 token and block matching), four denoising
    steps: the first cold, the rest warm, against the uncached block."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import BlockRunner, FullBlockRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    K = args.cfg_steps
    out = {}
    for name in ("latte_block", "svdxt_block"):
        if args.only and args.only != name:
            continue
        wl = make_workload(name, 4)
        xs = [_bf16_dev(s, dev) for s in wl.steps]
        Ws = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
        Wt = {k: _bf16_dev(v, dev) for k, v in wl.t_weights.items()}
        shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, 0, "bf16")
        cs = oc.Cfg(wl.gran, r=wl.r, r_frame=wl.r_frame, patch_k=wl.patch_k)
        ct = oc.Cfg("block", r=wl.extra["r_block"], patch_k=wl.extra["block_patch_k"])
        full = FullBlockRunner(shape, Ws, Wt, dev)
        full_ms = timed_ms(full, xs, K, 3)
        run = BlockRunner(shape, cs, ct, Ws, Wt, dev)
        # the four-step chain, each step timed alone (the first is cold)
        chain_us = []
        for rep in range(3):
            run.reset()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
            torch.cuda.synchronize()
            e[0].record()
            for s in range(4):
                run(xs[s])
                e[s + 1].record()
            torch.cuda.synchronize()
            chain_us.append([e[i].elapsed_time(e[i + 1]) * 1e3 for i in range(4)])
        steps_us = [round(sorted(c[i] for c in chain_us)[1], 2) for i in range(4)]
        warm_ms = timed_ms(run, xs[1:], K, 3)
        stages = stage_times(run, xs[1:], K)
        kernels = {k: dict(avg_us=round(v[0] * 1e3 / max(v[1], 1), 3), launches_per_step=round(v[1] / K, 3))
                   for k, v in stages.items()}
        ps, pt = oc.plan(shape, cs), oc.plan(shape, ct)
        out[name] = dict(
            workload=f"F={wl.F}, {wl.H}x{wl.W} tokens, C={wl.C}, {wl.heads}x{wl.head_dim}, bf16; spatial "
                     f"{wl.gran} r_f={wl.r_frame} r_t={wl.r} k={wl.patch_k}, temporal block r_b="
                     f"{wl.extra['r_block']} k={wl.extra['block_patch_k']}",
            steps_us=steps_us, warm_us=round(warm_ms * 1e3, 2), uncached_us=round(full_ms * 1e3, 2),
            speedup_warm=round(full_ms / warm_ms, 4),
            speedup_4_steps=round(4 * full_ms * 1e3 / sum(steps_us), 4),
            spatial_retained=f"{ps.n_seq}x{ps.seq_len}", temporal_retained=f"{pt.n_seq}x{pt.seq_len}",
            kernels=kernels)
        del run, full, xs, Ws, Wt
        torch.cuda.empty_cache()
    return out


def run_k_sweep(args):
    """Token-group count at the SD3-like shape (k x k patches, k = 1, 2, 4, 8:
    1 to 64 groups per frame, §3.3 and App. A's group counts): the step and
    its bookkeeping kernels (norms, similarity, selection) and the standalone
    gather and restore entry points, r = 0.5."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import LayerRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    K = args.cfg_steps
    wl = make_workload("sd3_1024", 3)
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, wl.n_ctx, "bf16")
    xs = [_bf16_dev(s, dev) for s in wl.steps]
    W = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
    ctx = _bf16_dev(wl.ctx, dev)
    out = {}
    for k in (1, 2, 4, 8):
        cfg = oc.Cfg("token", r=0.5, patch_k=k)
        run = LayerRunner(shape, cfg, W, dev, ctx)
        run(xs[0])
        ms = timed_ms(run, xs[1:], K, 3)
        st = stage_times(run, xs[1:], K)
        pl = oc.plan(shape, cfg)
        _, _, tr = oc.layer_cached(xs[1], W, run.cache, shape, cfg, ctx=ctx, ws=run.ws, trace=True)
        kept, rmap = tr["kept_idx"], tr["restore_map"]
        y_kept = torch.empty((kept.numel(), shape.C), dtype=torch.bfloat16, device=dev)
        y_out = torch.empty_like(run.cache.y)
        mv = stage_times(lambda _x: (oc.gather(xs[2], kept, shape, cfg),
                                     oc.restore(y_kept, rmap, shape, cache_y=y_out, y=y_out)), [None], K)

        def us(d, name):
            return round(d[name][0] * 1e3 / max(d[name][1], 1), 3) if name in d else None

        out[str(k)] = dict(groups=pl.n_groups, candidates_per_group=pl.n_src_max, reps_per_group=pl.n_dst_max,
                           step_us=round(ms * 1e3, 2), inv_norm_us=us(st, "inv_norm"), match_us=us(st, "match"),
                           select_us=us(st, "select"), compact_us=us(st, "compact"),
                           gather_us=us(mv, "gather"), restore_us=us(mv, "restore"),
                           match_gflop=round(2.0 * pl.n_groups * pl.n_src_max * pl.n_dst_max * wl.C / 1e9, 3))
        del run
    return out


def run_two_level(args):
    """The hierarchy of §3.3 at the SD3-like shape: Token Cache matched in
    k x k patches first, then in coarser patches or the whole frame among the
    candidates left, against one level at the same total ratio (r = 0.5):
    the step, the uncached layer, and the bookkeeping stages."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import FullRunner, LayerRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    K = args.cfg_steps
    wl = make_workload("sd3_1024", 3)
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, wl.n_ctx, "bf16")
    xs = [_bf16_dev(s, dev) for s in wl.steps]
    W = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
    ctx = _bf16_dev(wl.ctx, dev)
    full_ms = timed_ms(FullRunner(shape, oc.Cfg("token", 0.0), W, dev, ctx), xs, K, 3)
    out = dict(uncached_us=round(full_ms * 1e3, 2))
    for name, cfg in (("one level, k=1, r=0.5", oc.Cfg("token", r=0.5)),
                      ("one level, k=4, r=0.5", oc.Cfg("token", r=0.5, patch_k=4)),
                      ("k=4 r=0.25, then k=1 r=0.25", oc.Cfg("token", r=0.25, patch_k=4, coarse_k=1, r_coarse=0.25)),
                      ("k=8 r=0.25, then k=2 r=0.25", oc.Cfg("token", r=0.25, patch_k=8, coarse_k=2, r_coarse=0.25)),
                      ("k=4 r=0.4, then k=1 r=0.1", oc.Cfg("token", r=0.4, patch_k=4, coarse_k=1, r_coarse=0.1))):
        run = LayerRunner(shape, cfg, W, dev, ctx)
        run(xs[0])
        ms = timed_ms(run, xs[1:], K, 3)
        st = stage_times(run, xs[1:], K)
        book = ("inv_norm", "match", "select", "compact", "fill")
        pl = oc.plan(shape, cfg)
        out[name] = dict(step_us=round(ms * 1e3, 2), speedup_vs_uncached=round(full_ms / ms, 4),
                         retained_tokens=pl.n_kept,
                         bookkeeping_us=round(sum(st[n][0] for n in book if n in st) * 1e3 / K, 3),
                         stages_us={n: round(v[0] * 1e3 / K, 3) for n, v in st.items()})
        del run
    return out


def run_frame_patch_sweep(args):
    """Frame Cache scope on the Latte-like spatial layer (§3.3): whole-frame
    matching (k = 1) against per-patch matching on 2x2 and 4x4 patches
    (k = 2, 4; frames then keep varying numbers of tokens), r_f = 0.25: the
    step, its matching-stage kernels and the retained token count."""
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import LayerRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    K = args.cfg_steps
    wl = make_workload("latte_spatial", 3)
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, 0, "bf16")
    xs = [_bf16_dev(s, dev) for s in wl.steps]
    W = {k: _bf16_dev(getattr(wl, k), dev) for k in ("wq", "wk", "wv", "wo")}
    out = {}
    for k in (1, 2, 4):
        cfg = oc.Cfg("frame", r_frame=0.25, patch_k=k)
        run = LayerRunner(shape, cfg, W, dev)
        run(xs[0])
        ms = timed_ms(run, xs[1:], K, 3)
        st = stage_times(run, xs[1:], K)
        match_stages = ("frame_gram", "frame_reduce", "frame_final", "inv_norm", "match", "select", "compact")
        out[str(k)] = dict(groups=oc.plan(shape, cfg).n_groups, step_us=round(ms * 1e3, 2),
                           matching_us=round(sum(st[n][0] for n in match_stages if n in st) * 1e3 / K, 3),
                           stages_us={n: round(v[0] * 1e3 / max(v[1], 1), 3) for n, v in st.items()},
                           retained_tokens=oc.plan(shape, cfg).n_kept)
        del run
    return out


def run_layered(args):
    """Layered Cache schedule proposal (Alg. 1) on SD3-shaped synthetic
    tables (24 blocks x 28 steps): host time of oc_layered_schedule and the
    schedule it returns at the paper's SD3 speed-ups."""
    import paper_2607_23844_amd as oc
    from oc_synth import layered_tables
    lat, qual = layered_tables()
    out = {}
    for s_r in (1.2, 1.35, 1.75, 2.32):
        t0 = time.perf_counter()
        for _ in range(20):
            chosen, saved, budget = oc.layered_schedule(lat, qual, s_r, 2)
        dt = (time.perf_counter() - t0) / 20
        out[str(s_r)] = dict(pairs_cached=len(chosen), of_pairs=int(lat.size), saved=round(saved, 4),
                             budget=round(budget, 4), host_us=round(dt * 1e6, 1))
    return out


def run_data_movement_svdxt(args):
    """The gather and restore entry points at the SVD-XT-like level (25
    frames of 9216 tokens, C = 320, 92160 retained rows): large enough for
    HBM bandwidth rather than launch latency to set their time."""
    import numpy as np
    import torch
    import paper_2607_23844_amd as oc
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    wl = make_workload("svdxt_level", 2)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(dev)

    xs = [t(s) for s in wl.steps]
    W = {k: t(getattr(wl, k)) for k in ("wq", "wk", "wv", "wo")}
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, 0, "bf16")
    cfg = oc.Cfg(wl.gran, r=wl.r, r_frame=wl.r_frame, patch_k=wl.patch_k)
    res = run_data_movement(args, shape, cfg, W, xs, None)
    del xs, W
    torch.cuda.empty_cache()
    return res


def run_data_movement(args, shape, cfg, W, xs, ctx):
    """The standalone gather and (in-place) restore entry points: kernel time
    and HBM GB/s (2 n_kept C bytes-per-element moved) with warm caches, after
    a 512 MiB write that flushes L2 and MALL ("flushed": the dirty lines it
    leaves are written back during the measured kernel), and after a 512 MiB
    read ("flushed_read": the caches hold clean, unrelated lines)."""
    import torch
    import paper_2607_23844_amd as oc

    dev = xs[0].device
    cache = oc.LayerCache(shape, dev)
    y, _, tr = oc.layer_cached(xs[0], W, cache, shape, cfg, ctx=ctx, trace=True)
    kept, rmap = tr["kept_idx"], tr["restore_map"]
    y_kept = torch.empty((kept.numel(), shape.C), dtype=xs[0].dtype, device=dev)
    y_out = torch.empty_like(cache.y)
    flush = torch.empty(512 << 20, dtype=torch.uint8, device=dev)
    nbytes = 2.0 * kept.numel() * shape.C * 2
    res = {}
    for name, fn in (("gather", lambda: oc.gather(xs[1], kept, shape, cfg)),
                     ("restore", lambda: oc.restore(y_kept, rmap, shape, cache_y=y_out, y=y_out))):
        for mode in ("warm", "flushed", "flushed_read"):
            timer = oc.StageTimer()
            for i in range(args.cfg_steps + 3):
                if mode == "flushed":
                    flush.zero_()
                elif mode == "flushed_read":
                    flush_sum = flush.view(torch.int32).sum()   # noqa: F841 (reads every line)
                if i == 3:
                    timer.reset()
                with timer:
                    fn()
            torch.cuda.synchronize()
            st = timer.collect()
            tot, n = st[name]
            us = tot * 1e3 / max(n, 1)
            res[f"{name}_{mode}"] = dict(avg_us=round(us, 3), gbs=round(nbytes / (us * 1e-6) / 1e9, 1),
                                         frac_hbm=round(nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS, 4))
    # the same moves by torch's own kernels (index_select: a gather of the
    # rows; index_copy_: the row scatter a kept-list restore would do), each
    # call and the library's entry points alike timed by events around it,
    # median of 10; a short spin kernel queued first keeps the GPU busy while
    # the host queues the events and the call, so the host's launch time
    # stays out of the interval
    keptl = kept.long()
    x2, y2 = xs[1].view(-1, shape.C), y_out.view(-1, shape.C)
    vendor = {}
    for name, fn in (("oc_gather", lambda: oc.gather(xs[1], kept, shape, cfg)),
                     ("torch_index_select", lambda: torch.index_select(x2, 0, keptl)),
                     ("oc_restore", lambda: oc.restore(y_kept, rmap, shape, cache_y=y_out, y=y_out)),
                     ("torch_index_copy", lambda: y2.index_copy_(0, keptl, y_kept))):
        for mode in ("warm", "flushed", "flushed_read"):
            ts = []
            for i in range(13):
                if mode == "flushed":
                    flush.zero_()
                elif mode == "flushed_read":
                    flush_sum = flush.view(torch.int32).sum()   # noqa: F841
                torch.cuda._sleep(100000)
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                fn()
                e1.record()
                torch.cuda.synchronize()
                if i >= 3:
                    ts.append(e0.elapsed_time(e1) * 1e3)
            vendor[f"{name}_{mode}_us"] = round(statistics.median(ts), 1)
    res["event_timed_vs_torch"] = vendor
    res["bytes_per_call"] = nbytes
    return res


def achievable_peaks():
    """What vendor code reaches on this machine, beside the spec peaks the
    roofline uses: a bf16 GEMM of 8192 x 8192 x 8192 through torch.matmul
    (hipBLASLt), the same GEMM at the SD3-like layer's shapes, and a 1 GiB
    device-to-device copy (read + write bytes)."""
    import torch
    dev = torch.device("cuda:0")

    def best(fn, reps=10):
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e-3 / reps

    n = 8192
    a = torch.randn((n, n), device=dev).to(torch.bfloat16)
    b = torch.randn((n, n), device=dev).to(torch.bfloat16)
    c = torch.empty((n, n), device=dev, dtype=torch.bfloat16)
    t_mm = best(lambda: torch.matmul(a, b, out=c))
    del a, b, c
    src = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    dst = torch.empty_like(src)
    t_cp = best(lambda: dst.copy_(src))
    del src, dst
    # the same vendor GEMM at the SD3-like layer's own shapes (r = 0.5:
    # 2381 attention rows; the similarity at k = 1 without its arg-max)
    same_shape = {}
    for name, (m, nn, k) in (("similarity_3072x1024x1536", (3072, 1024, 1536)),
                             ("qk_projection_2381x3072x1536", (2381, 3072, 1536)),
                             ("qkv_projection_2381x4608x1536", (2381, 4608, 1536)),
                             ("v_or_out_projection_2381x1536x1536", (2381, 1536, 1536))):
        a = torch.randn((m, k), device=dev).to(torch.bfloat16)
        b = torch.randn((nn, k), device=dev).to(torch.bfloat16)
        c = torch.empty((m, nn), device=dev, dtype=torch.bfloat16)
        t = best(lambda: torch.matmul(a, b.t(), out=c), reps=50)
        same_shape[name] = dict(us=round(t * 1e6, 2), tflops=round(2.0 * m * nn * k / t / 1e12, 1))
        del a, b, c
    torch.cuda.empty_cache()
    mm = 2.0 * n ** 3 / t_mm / 1e12
    cp = 2.0 * (1 << 30) / t_cp / 1e9
    return dict(mfma_bf16_tflops=round(mm, 1), mfma_frac_of_spec=round(mm / PEAK_MFMA_TFLOPS, 4),
                mfma_source="torch.matmul bf16 8192^3 (hipBLASLt)", hbm_gbs=round(cp, 1),
                hbm_frac_of_spec=round(cp / PEAK_HBM_GBS, 4), hbm_source="torch copy_ of 1 GiB (read + write)",
                vendor_gemm_at_layer_shapes=same_shape)


def run_gpu(args):
    import numpy as np
    import torch
    import paper_2607_23844_amd as oc
    from paper_2607_23844_amd.runner import FullRunner, LayerRunner
    from oc_synth import make_workload

    dev = torch.device("cuda:0")
    wl = make_workload("sd3_1024", 4)
    shape = oc.Shape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, wl.n_ctx, "bf16")

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(dev)

    xs = [t(s) for s in wl.steps]
    ctx = t(wl.ctx)
    W = {k: t(getattr(wl, k)) for k in ("wq", "wk", "wv", "wo")}
    tokens = shape.F * shape.N + shape.n_ctx
    K, Wm = args.steps, args.warmup

    def timed(fn, inputs):
        for i in range(Wm):
            fn(inputs[i % len(inputs)])
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0 = time.perf_counter()
        e0.record()
        for i in range(K):
            fn(inputs[i % len(inputs)])
        e1.record()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        return e0.elapsed_time(e1) / K, wall

    full = FullRunner(shape, oc.Cfg("token", 0.0), W, dev, ctx)
    full_ms, _ = timed(full, xs)
    by_r = {}
    primary = None
    for r in sorted(set([0.25, 0.5, 0.75, args.r])):
        cfg = oc.Cfg("token", r=r, patch_k=1)
        run = LayerRunner(shape, cfg, W, dev, ctx)
        run(xs[0])                       # cold step: the layer cache becomes valid
        ms, wall = timed(run, xs[1:])
        by_r[str(r)] = dict(ms=ms, tokens_per_s=tokens / (ms * 1e-3), speedup_vs_uncached=full_ms / ms)
        if r == args.r:
            primary = (cfg, run, ms, wall)
        else:
            # the other ratios' stages, live time per step (µs)
            rs = stage_times(run, xs[1:4], K)
            by_r[str(r)]["stages_us"] = {st: round(t * 1e3 / K, 2) for st, (t, n) in rs.items()}
    cfg, run, ms, wall = primary
    pct = step_percentiles(run, xs[1:], K)
    graph_us = graph_latency(run, xs[1], K)
    clock = sampled_clock(run, xs[1:])
    moves = run_data_movement(args, shape, cfg, W, xs, ctx)
    # (the per-kernel loop below is the last use of these kernels at this
    # shape, so a profiler trace can pick out exactly its launches)
    # live per-kernel timing: HIP events stamped by the runtime at each kernel's start and end
    stages = stage_times(run, xs[1:4], K)
    pl = oc.plan(shape, cfg)
    kernels, roof = kernel_table(stages, K, stage_work(shape, cfg, pl, shape.n_ctx), "sd3_1024")
    del run, full
    torch.cuda.empty_cache()
    peaks = achievable_peaks()
    return dict(ms=ms, wall=wall, tokens=tokens, full_ms=full_ms, by_r=by_r, kernels=kernels, roofline=roof,
                plan=dict(n_kept=pl.n_kept, n_cached=pl.n_cached, seq_len=pl.seq_len), pct=pct, graph_us=graph_us,
                moves=moves, peaks=peaks, clock=clock)


def sampled_clock(fn, inputs, n=4000, gap=50):
    """The shader clock while the step runs: the library's one-wave sampler
    (oc_clock_sample) on a second stream takes n readings gap / 100 µs
    apart (2 ms) while 30 steps run on the current stream, after the timed
    region; the same sampler alone gives the idle clock.  GHz p10 / p50 /
    p90 over the intervals."""
    import numpy as np
    import torch
    import paper_2607_23844_amd as oc
    dev = torch.device("cuda:0")
    buf = torch.zeros(2 * n, dtype=torch.int64, device=dev)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    oc.clock_sample(buf, n, gap, side)
    torch.cuda.synchronize()
    idle = float(np.median(oc.clock_ghz(buf)))
    oc.clock_sample(buf, n, gap, side)
    steps = 30                          # about 4.5 ms of steps: past the whole sampling window
    for i in range(steps):
        fn(inputs[i % len(inputs)])
    torch.cuda.synchronize()
    q = np.percentile(oc.clock_ghz(buf), [10, 50, 90])
    return dict(idle=round(idle, 3), p10=round(float(q[0]), 3), p50=round(float(q[1]), 3),
                p90=round(float(q[2]), 3), steps=steps, window_us=n * gap / 100.0)


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or platform.machine()


def run_cpu_baselines(args):
    """The CPU oracle, unchanged, on one thread pinned to one core: a cold step
    (no layer cache) and a warm step of each workload, the median of three
    runs (C1-C4).  The SVD-XT-sized level (C5) is timed on a bounded sample:
    its decisions in full (patch-local matching, k = 4), then the attention
    of one of its sequences, scaled to all of them.  The headline figure is
    the SD3-like layer's warm step."""
    import statistics
    from threadpoolctl import threadpool_limits
    from oc_synth import make_workload
    from oracle import oc_oracle as O

    try:
        os.sched_setaffinity(0, {sorted(os.sched_getaffinity(0))[-1]})
        pinned = True
    except (AttributeError, OSError):
        pinned = False
    out = {}
    reps = args.cpu_reps
    with threadpool_limits(1):
        for key, name in (("C1_tok16_f32", "tok16_f32"), ("C2_sd3_1024", "sd3_1024"),
                          ("C3_latte_spatial", "latte_spatial"), ("C4_latte_temporal", "latte_temporal")):
            wl = make_workload(name, 2)
            sh = O.LayerShape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim, wl.n_ctx)
            cf = O.CacheCfg(wl.gran, r=wl.r, r_frame=wl.r_frame, patch_k=wl.patch_k)
            W = {k: wl.f64(getattr(wl, k)) for k in ("wq", "wk", "wv", "wo")}
            ctx = wl.f64(wl.ctx) if wl.n_ctx else None
            x0, x1 = wl.f64(wl.steps[0]), wl.f64(wl.steps[1])
            cold, warm = [], []
            for _ in range(reps):
                t0 = time.perf_counter()
                r0 = O.layer_step(x0, ctx, W, sh, cf, None, False)
                t1 = time.perf_counter()
                O.layer_step(x1, ctx, W, sh, cf, r0.y, True)
                t2 = time.perf_counter()
                cold.append(t1 - t0)
                warm.append(t2 - t1)
            tokens = wl.F * wl.N + wl.n_ctx
            c, w = statistics.median(cold), statistics.median(warm)
            out[key] = dict(cold_s=round(c, 4), warm_s=round(w, 4), tokens_per_s=round(tokens / w, 2),
                            runs=reps, tokens_per_step=tokens)
        # C5: bounded sample
        wl = make_workload("svdxt_level_k4", 2)
        sh = O.LayerShape(wl.F, wl.H, wl.W, wl.C, wl.heads, wl.head_dim)
        cf = O.CacheCfg(wl.gran, r=wl.r, r_frame=wl.r_frame, patch_k=wl.patch_k)
        W = {k: wl.f64(getattr(wl, k)) for k in ("wq", "wk", "wv", "wo")}
        x = wl.f64(wl.steps[1]).reshape(wl.F, wl.N, wl.C)
        t0 = time.perf_counter()
        dec = O.decide(x, sh, cf)
        seqs = O.build_sequences(sh, cf, dec)
        kept, _, rmap = O.kept_and_map(sh, cf, dec, seqs, True)
        t1 = time.perf_counter()
        X = x.reshape(-1, wl.C)[seqs[0]]
        O.multi_head_attention(X, W["wq"], W["wk"], W["wv"], W["wo"], wl.heads, wl.head_dim)
        t2 = time.perf_counter()
        step = (t1 - t0) + len(seqs) * (t2 - t1)
        tokens = wl.F * wl.N
        out["C5_svdxt_level_k4"] = dict(
            warm_s_estimated=round(step, 3), tokens_per_s=round(tokens / step, 2), decisions_s=round(t1 - t0, 3),
            one_sequence_s=round(t2 - t1, 3), sequences=len(seqs),
            sample="decisions in full (frame stage, pairing, token matching in 4x4 patches, selection, maps), then "
                   f"the attention of 1 of the {len(seqs)} sequences of {len(seqs[0])} tokens, scaled to all; the "
                   "cold step differs only in its restore map (the same work)")
    head = out["C2_sd3_1024"]
    return dict(value=head["tokens_per_s"], unit="tokens/s", cores=1, kind="oracle",
                sample=f"median of {reps} warm steps of the full SD3-like layer (4096+333 tokens, r=0.5), fp64 NumPy, "
                       f"one thread{' pinned to one core' if pinned else ''}; {head['warm_s']:.2f} s per step; "
                       f"1 of {os.cpu_count()} logical CPUs of the host ({_cpu_model()})",
                configs=out)


ONLY = ("sd3_1024", "latte_spatial", "latte_temporal", "svdxt_level", "svdxt_level_k4", "sd3_ffn", "latte_block",
        "svdxt_block", "k_sweep", "two_level")


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--r", type=float, default=0.5)
    ap.add_argument("--cpu-reps", type=int, default=3, help="runs of each CPU oracle step (median)")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baselines")
    ap.add_argument("--cfg-steps", type=int, default=20, help="timed steps per additional configuration")
    ap.add_argument("--no-configs", action="store_true",
                    help="skip everything but the SD3-like layer (Latte, SVD-XT, FFN, blocks, group sweep)")
    ap.add_argument("--only", choices=ONLY, default=None,
                    help="run one workload's GPU measurement alone and print its result (for per-workload profiles)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="first run a plain 256 MiB read + 256 MiB write elementwise kernel (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on exactly one GPU: the cached layer is measured whole on a single MI355X and there is "
              f"no multi-GPU path (asked for --gpus {args.gpus})", file=sys.stderr)
        sys.exit(2)
    if args.copy_probe:
        import torch
        src = torch.ones(64 << 20, dtype=torch.float32, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.mul(src, 1.0, out=dst)
        torch.cuda.synchronize()
        del src, dst
    if args.only and args.only != "sd3_1024":
        fn = {"sd3_ffn": run_ffn, "latte_block": run_blocks, "svdxt_block": run_blocks, "k_sweep": run_k_sweep,
              "two_level": run_two_level}.get(
            args.only, run_other_configs)
        print(json.dumps({"only": args.only, "result": fn(args)}))
        return
    g = run_gpu(args)
    extra = {}
    if not args.no_configs and not args.only:
        extra["other_configs"] = run_other_configs(args)
        g["moves"]["svdxt_level"] = run_data_movement_svdxt(args)
        extra["ffn_sd3"] = run_ffn(args)
        extra["blocks"] = run_blocks(args)
        extra["group_count_sweep_sd3"] = run_k_sweep(args)
        extra["two_level_hierarchy_sd3"] = run_two_level(args)
        extra["frame_patch_sweep_latte"] = run_frame_patch_sweep(args)
        extra["layered_schedule"] = run_layered(args)
    cpu = None if (args.no_cpu or args.only) else run_cpu_baselines(args)
    ms = g["ms"]
    line = {
        "metric": METRIC,
        "value": round(g["tokens"] / (ms * 1e-3), 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {
            "workload": f"SD3-1024-like joint-attention layer, Token Cache r={args.r}: F=1, 64x64 image tokens + "
                        f"333 uncached text tokens, C=1536, 24 heads x 64, bf16, patch_k=1, warm layer cache",
            "r": args.r,
            "tokens_per_step": g["tokens"],
            "retained_image_tokens": g["plan"]["n_kept"],
        },
        "latency_us": round(ms * 1e3, 2),
        "latency_pct_us": g["pct"],
        "graph_latency_us": g["graph_us"]["graph_us"],
        "graph_vs_eager_interleaved_us": g["graph_us"],
        "clock_under_load_ghz": g["clock"],
        "uncached_latency_us": round(g["full_ms"] * 1e3, 2),
        "speedup_vs_uncached": round(g["full_ms"] / ms, 4),
        "by_r": {k: {kk: (round(vv, 4) if isinstance(vv, float) else vv) for kk, vv in v.items()}
                 for k, v in g["by_r"].items()},
        "roofline": g["roofline"],
        "kernels": g["kernels"],
        "data_movement": g["moves"],
        **extra,
        "achievable_peaks": g["peaks"],
        "paper_context": "model-level latency cuts of up to 35% / 25% / 28% (SD3 / SVD-XT / Latte) on one A100 40 GB, "
                         "precision not stated; no per-layer figure is published",
        "cpu_baseline": cpu,
        "wall_s_timed_region": round(g["wall"], 4),
    }
    print(json.dumps(line))


if __name__ == "__main__":
    main()
