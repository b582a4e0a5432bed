#!/usr/bin/env python3
"""Throughput of the fused Compactor hot path (score -> select -> compact) on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 2] [--group-mb M]

A step is one compactor_compress call over the whole synthetic batch, inputs already
resident in HBM.  Prints ONE JSON line: tokens compressed per second, the roofline of the
dominant kernel (algorithmic bytes / its HIP-event duration, against the 8 TB/s HBM peak) and
the float64 CPU oracle timed on a bounded sample of the same workload as a reported baseline.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# HBM bytes per launch measured with rocprofv3 (FETCH_SIZE x 2.000 + WRITE_SIZE x 1.000, the
# scale factors read off a 1 GiB copy kernel), by (workload, mode, kernel):
# profiles/compress_config*_hbm_traffic.txt.  Workloads that have not been profiled report null.
MEASURED_TRAFFIC_BYTES = {
    ("config2_llama31_8b_n32768", "sketched", "gather"): 2.607e9,
    ("config2_llama31_8b_n32768", "sketched", "gram"): 2.169e9,
    ("config2_llama31_8b_n32768", "sketched", "score"): 2.232e9,
    ("config3_qwen25_7b_n131072", "sketched", "gather"): 3.041e9,
    ("config3_qwen25_7b_n131072", "sketched", "gram"): 3.783e9,
    ("config3_qwen25_7b_n131072", "sketched", "score"): 3.842e9,
    ("config4_ragged_batch", "sketched", "gather"): 6.558e10,
    ("config4_ragged_batch", "sketched", "gram"): 4.335e10,
    ("config4_ragged_batch", "sketched", "score"): 4.458e10,
    ("config5_qwen25_32b_n100000", "sketched", "gather"): 1.691e10,
    ("config5_qwen25_32b_n100000", "sketched", "gram"): 1.313e10,
    ("config5_qwen25_32b_n100000", "sketched", "score"): 1.342e10,
    ("config5_qwen25_32b_n100000", "exact,", "gather"): 1.691e10,
    ("config5_qwen25_32b_n100000", "exact,", "gram"): 1.313e10,
    ("config5_qwen25_32b_n100000", "exact,", "score"): 1.349e10,
}
HBM_PEAK_GBS = 8000.0           # MI355X published HBM3E bandwidth
MFMA_BF16_PEAK_TFLOPS = 2500.0  # MI355X published dense bf16 MFMA rate


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=int(os.environ.get("WORLD_SIZE", "1")))
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=4, choices=[1, 2, 3, 4, 5],
                    help="headline workload (default: config 4, the largest that runs on one GPU)")
    ap.add_argument("--exact", action="store_true",
                    help="exact leverage scores (no sketch) with ridge_rel 1e-4: config 5's second mode")
    ap.add_argument("--only", action="store_true",
                    help="time the headline workload only (no `configs` array of the other workloads)")
    ap.add_argument("--layers", type=int, default=0, help="override the layer count (0 = config's own)")
    ap.add_argument("--group-mb", type=float, default=0.0, help="head-group size in MiB (0 = library default)")
    ap.add_argument("--gram-wgs", type=int, default=0, help="tuning override (0 = library's choice)")
    ap.add_argument("--score-tokens", type=int, default=0, help="tuning override (0 = library's choice)")
    ap.add_argument("--scope", choices=["head", "layer"], default="head",
                    help="selection pool: per head (the headline metric) or head-adaptive per layer")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one 1 GiB device-to-device copy (a dispatch of known size against "
                         "which rocprofv3's FETCH_SIZE / WRITE_SIZE counters are scaled)")
    ap.add_argument("--attention", action="store_true",
                    help="measure compactor_attention_scores (Sec. 3.2 scores a) and the blended "
                         "compress on the same workload instead of the default line")
    ap.add_argument("--q-per-kv", type=int, default=4, help="query heads per kv head for --attention")
    ap.add_argument("--paged", action="store_true",
                    help="time the compaction stage with a paged destination (and in place)")
    ap.add_argument("--page-size", type=int, default=16, help="slots per page for --paged")
    ap.add_argument("--graph", action="store_true",
                    help="also capture one step in a HIP graph and time its replays (graph_ms_per_step)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="time budget of each oracle leg")
    ap.add_argument("--cpu-threads", type=int, default=0,
                    help="cap the oracle leg's BLAS threads (0 = the host's default, all cores)")
    ap.add_argument("--flush-cache", action="store_true",
                    help="also time steps one by one, each after a 512 MiB fill that evicts the "
                         "last-level cache (cold_ms_per_step); matters for workloads that fit in it")
    return ap.parse_args()


def build_workload(W, cfg, dev, layers, exact=False):
    kw = {"device": dev}
    if layers:
        kw["L"] = layers
    w = {1: W.config1, 2: W.config2, 3: W.config3, 4: W.config4, 5: W.config5}[cfg](**kw)
    if exact:
        w.sketch_dim, w.ridge_rel = 0, 1e-4
    return w


# algorithmic HBM bytes per head-row of each stage (d = 128, bf16 K/V, fp32 scores, int32 idx)
def stage_bytes(w, kk):
    LH = w.layers * w.kv_heads
    rows = sum(r.n for r in w.requests) * LH
    kept = sum(k for k in kk) * LH
    return {
        "gram": 256.0 * rows,                 # K read once
        "score": 260.0 * rows,                # K read again + fp32 score written
        "select": 8.0 * rows,                 # scores read (histogram + emit)
        "gather": 1028.0 * kept,              # 4-byte index, K and V rows read and written
        # (the index is counted once, with the stage that consumes it: 524 + 1028 r in all)
    }, rows, kept


def stage_flops(w, ks):
    LH = w.layers * w.kv_heads
    rows = sum(r.n for r in w.requests) * LH
    m = ks if ks > 0 else 128
    return {"gram": 2.0 * 128 * 128 * rows, "score": 2.0 * 128 * m * rows}


def cpu_baseline(W, O, w, phi, budget_s, threads=0):
    """The oracle as it stands on the host cores, on as many heads of the workload as fit the
    time budget (at least one), scaled linearly to all heads (heads are independent)."""
    import numpy as np
    from threadpoolctl import threadpool_info, threadpool_limits
    if threads > 0:
        with threadpool_limits(limits=threads):
            return cpu_baseline(W, O, w, phi, budget_s)
    cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    LH = w.layers * w.kv_heads
    phi_np = phi.double().cpu().numpy() if phi is not None else None
    t_total, done, head_rows = 0.0, 0, 0
    for b, r in enumerate(w.requests):
        for g in range(LH):
            l, h = divmod(g, w.kv_heads)
            kb = W.bf16_bits(r.k[l, h])
            vb = W.bf16_bits(r.v[l, h])
            t0 = time.perf_counter()
            K = O.bf16_bits_to_f64(kb)
            O.compress_head(K, kb, vb, r.ratio, phi_np, w.ridge_rel, None, W.LAMBDA_BLEND)
            t_total += time.perf_counter() - t0
            done += 1
            head_rows += r.n
            if t_total >= budget_s:
                break
        if t_total >= budget_s:
            break
    rows_per_s = head_rows / t_total
    tokens_per_s = rows_per_s / LH          # a token carries L*H head-rows
    return {"value": tokens_per_s, "unit": "tokens/s", "cores": int(cores), "kind": "oracle",
            "sample": "%d of %d heads (%d head-rows) in %.1f s, scaled linearly in heads" %
                      (done, LH * len(w.requests), head_rows, t_total)}


def attention_mode(a, torch, C, W, w, reqs, params, bufs, dev):
    """Times the attention-score kernels alone and the full Compactor step (a, then the fused
    compress with the blend), on the same synthetic keys plus synthetic queries."""
    G = a.q_per_kv
    ap = C.AttnParams(w.layers, w.kv_heads, w.kv_heads * G)
    qs = [W.synthetic_queries(w.layers, w.kv_heads * G, r.n, device=dev, request=i) for i, r in enumerate(w.requests)]
    areqs = [C.AttnRequest(q, r.k) for q, r in zip(qs, w.requests)]
    total = sum(w.layers * w.kv_heads * r.n for r in w.requests)
    attn = torch.empty(total, dtype=torch.float32, device=dev)
    aws = torch.empty(max(256, C.compactor_attention_workspace_size(ap, areqs)), dtype=torch.uint8, device=dev)
    off, breqs = 0, []
    for r in w.requests:
        cnt = w.layers * w.kv_heads * r.n
        breqs.append(C.Request(k_score=r.k, v_cache=r.v, ratio=r.ratio, attn=attn[off:off + cnt]))
        off += cnt

    def run(fn):
        for _ in range(a.warmup):
            fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(a.steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / a.steps * 1e3

    ms_attn = run(lambda: C.compactor_attention_scores(ap, areqs, attn=attn, workspace=aws))
    # the blended compress needs a little more workspace than the plain one (the blend's sums)
    bufs = dict(bufs)
    bufs["workspace"] = torch.empty(max(256, C.compactor_workspace_size(params, breqs)), dtype=torch.uint8, device=dev)
    ms_full = run(lambda: (C.compactor_attention_scores(ap, areqs, attn=attn, workspace=aws),
                           C.compactor_compress(params, breqs, want_scores=False, **bufs)))
    # stage times of the blended compress (HIP events on the launch stream)
    ev = C.StageEvents()
    params.stage_events = ev
    stage_ms = {}
    for _ in range(a.steps):
        C.compactor_compress(params, breqs, want_scores=False, **bufs)
        torch.cuda.synchronize()
        for k_, v_ in ev.elapsed_ms().items():
            stage_ms[k_] = stage_ms.get(k_, 0.0) + v_ / a.steps
    params.stage_events = None
    rows_q = sum(r.n for r in w.requests) * w.layers * w.kv_heads * G
    rows_k = sum(r.n for r in w.requests) * w.layers * w.kv_heads
    flops = 2.0 * 256 * 128 * rows_q                   # Q K^T inside 256-token blocks
    nbytes = 256.0 * (rows_q + rows_k) + 8.0 * rows_k  # Q and K read once, sums written and pooled
    print(json.dumps({
        "metric": "attention scores a (Sec. 3.2) and full Compactor step at 1 GPU",
        "config": {"workload": w.name, "q_heads_per_kv_head": G, "chunk": 256, "pool": 7, "tokens": w.tokens},
        "attention_ms": ms_attn, "attention_TFLOP/s": flops / (ms_attn * 1e-3) / 1e12,
        "attention_GB/s": nbytes / (ms_attn * 1e-3) / 1e9,
        "attention_frac_of_8TB/s": nbytes / (ms_attn * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "attention_frac_of_bf16_mfma_peak": flops / (ms_attn * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS,
        "full_step_ms": ms_full, "full_step_tokens_per_s": w.tokens / (ms_full * 1e-3),
        "blended_compress_stages_ms": {k_: round(v_, 4) for k_, v_ in stage_ms.items()},
        "blend_GB/s": 16.0 * rows_k / (stage_ms.get("blend", float("nan")) * 1e-3) / 1e9,
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup, "dtype": "bf16", "data": "synthetic"}))


def paged_mode(a, torch, C, W, w, reqs, params, bufs, dev):
    """Times the compaction stage alone with a paged destination: dense source into pages, and in
    place inside the pages, beside the dense gather of the headline path."""
    ps = a.page_size
    C.compactor_compress(params, reqs, want_scores=False, **bufs)
    torch.cuda.synchronize()
    L, H = w.layers, w.kv_heads
    need = [(r.n + ps - 1) // ps for r in w.requests]
    num_pages = sum(need)
    g = torch.Generator(device="cpu")
    g.manual_seed(5)
    perm = torch.randperm(num_pages, generator=g).to(torch.int32).to(dev)   # scattered pages
    tables, at = [], 0
    for m in need:
        tables.append(perm[at:at + m].contiguous())
        at += m
    # one [pages, slot, head, d] pool per layer, seen as [page, layer, slot, head, d]
    kpool = torch.empty(L, num_pages, ps, H, 128, dtype=torch.bfloat16, device=dev)
    vpool = torch.empty_like(kpool)
    kview, vview = kpool.permute(1, 0, 2, 3, 4), vpool.permute(1, 0, 2, 3, 4)

    def fill():          # token t of every head at logical slot t
        for b, r in enumerate(w.requests):
            t = torch.arange(r.n, device=dev)
            pg, sl = tables[b].long()[t // ps], t % ps
            kview[pg, :, sl] = r.k.permute(2, 0, 1, 3)
            vview[pg, :, sl] = r.v.permute(2, 0, 1, 3)

    def timed(fn, before=None):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ms = []
        for i in range(a.warmup + a.steps):
            if before:
                before()
            e0.record()
            fn()
            e1.record()
            torch.cuda.synchronize()
            if i >= a.warmup:
                ms.append(e0.elapsed_time(e1))
        return sum(ms) / len(ms)

    ki, kc = bufs["kept_idx"], bufs["kept_cnt"]
    ms_dense = timed(lambda: C.compactor_compact(params, reqs, ki, kc, bufs["k_packed"], bufs["v_packed"]))
    ms_paged = timed(lambda: C.compactor_compact_paged(params, reqs, ki, kc, kview, vview, tables))
    steps = min(a.steps, 5)          # the refill is slow host-driven indexing
    a.steps, a.warmup = steps, 1
    ms_inplace = timed(lambda: C.compactor_compact_paged(params, reqs, ki, kc, kview, vview, tables,
                                                         in_place=True), before=fill)
    kept_rows = sum(L * H * C.compactor_keep_count(r.n, r.ratio) for r in w.requests)
    nbytes = 1028.0 * kept_rows
    print(json.dumps({
        "metric": "compaction stage with a paged destination at 1 GPU",
        "config": {"workload": w.name, "page_size": ps, "pages": num_pages, "kept_head_rows": kept_rows,
                   "select_scope": a.scope},
        "dense_ms": ms_dense, "dense_GB/s": nbytes / ms_dense / 1e6,
        "paged_ms": ms_paged, "paged_GB/s": nbytes / ms_paged / 1e6,
        "in_place_ms": ms_inplace, "in_place_GB/s": nbytes / ms_inplace / 1e6,
        "frac_of_8TB/s": {"dense": nbytes / ms_dense / 1e6 / HBM_PEAK_GBS,
                          "paged": nbytes / ms_paged / 1e6 / HBM_PEAK_GBS,
                          "in_place": nbytes / ms_inplace / 1e6 / HBM_PEAK_GBS},
        "n_gpus": 1, "dtype": "bf16", "data": "synthetic"}))


def measure(a, torch, C, W, w, dev, full=True):
    """Times the fused call on one workload.  -> dict with tokens/s, ms per step, per-stage event
    times, the dominant kernel's rate and the whole path's rate; with `full` also the unfused
    calls and the optional cold-cache and graph timings."""
    phi = W.make_phi(ks=w.sketch_dim, device=dev) if w.sketch_dim > 0 else None
    ev = C.StageEvents()
    group_bytes = int(a.group_mb * 1024 * 1024)
    mk = lambda events: C.Params(w.layers, w.kv_heads, sketch_dim=w.sketch_dim, phi=phi,
                                 ridge_rel=w.ridge_rel, group_bytes=group_bytes, stage_events=events,
                                 gram_wgs=a.gram_wgs, score_tokens=a.score_tokens,
                                 select_scope=(C.SCOPE_LAYER if a.scope == "layer" else C.SCOPE_HEAD))
    params, params_ev = mk(None), mk(ev)
    reqs = [C.Request(k_score=r.k, v_cache=r.v, ratio=r.ratio) for r in w.requests]
    so, ko, kk = C.compactor_layout(params, reqs)
    nh = len(reqs) * w.layers * w.kv_heads

    # every output and the workspace are allocated once, outside the timed region
    ws = torch.empty(max(256, C.compactor_workspace_size(params, reqs)), dtype=torch.uint8, device=dev)
    bufs = dict(kept_idx=torch.empty(ko[-1], dtype=torch.int32, device=dev),
                kept_cnt=torch.empty(nh, dtype=torch.int32, device=dev),
                k_packed=torch.empty(ko[-1], 128, dtype=torch.bfloat16, device=dev),
                v_packed=torch.empty(ko[-1], 128, dtype=torch.bfloat16, device=dev),
                status=torch.empty(nh, dtype=torch.int32, device=dev), workspace=ws)

    def step(p):
        C.compactor_compress(p, reqs, want_scores=False, **bufs)

    steps, warmup = (a.steps, a.warmup) if full else (max(3, a.steps // 2), max(1, a.warmup // 2))
    for _ in range(warmup):
        step(params)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step(params)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    ms_per_step = dt / steps * 1e3
    assert int(bufs["status"].max()) == 0, "a head was flagged during the benchmark"

    # the same steps again with per-stage HIP events on the launch stream
    stage_ms, step_ms = {}, []
    t1 = time.perf_counter()
    for _ in range(steps):
        step(params_ev)
        torch.cuda.synchronize()
        per = ev.elapsed_ms()
        step_ms.append(sum(per.values()))
        for k_, v_ in per.items():
            stage_ms[k_] = stage_ms.get(k_, 0.0) + v_ / steps
    ms_per_step_ev = (time.perf_counter() - t1) / steps * 1e3
    ms_median_ev = sorted(step_ms)[len(step_ms) // 2]   # first to last stage event, per step

    sbytes, rows, kept = stage_bytes(w, kk)
    sflops = stage_flops(w, w.sketch_dim)
    dominant = max(sbytes, key=lambda s: stage_ms.get(s, 0.0))
    achieved = sbytes[dominant] / (stage_ms[dominant] * 1e-3) / 1e9
    stages = {}
    for s_, ms in stage_ms.items():
        ent = {"ms": round(ms, 4)}
        if s_ in sbytes and ms > 0:
            ent["GB/s"] = round(sbytes[s_] / (ms * 1e-3) / 1e9, 1)
        if s_ in sflops and ms > 0:
            ent["TFLOP/s"] = round(sflops[s_] / (ms * 1e-3) / 1e12, 1)
        stages[s_] = ent
    total_bytes = sum(sbytes.values())
    mode = "sketched k_s=%d" % w.sketch_dim if w.sketch_dim > 0 else "exact, ridge_rel=%g" % w.ridge_rel
    res = {
        "workload": w.name, "mode": mode, "tokens": w.tokens, "head_rows": rows, "kept_head_rows": kept,
        "layers": w.layers, "kv_heads": w.kv_heads, "requests": len(reqs), "steps": steps,
        "value": w.tokens / (dt / steps), "ms_per_step": ms_per_step,
        "algorithmic_bytes": total_bytes,
        "path_frac_of_8TB/s": total_bytes / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "dominant_kernel": dominant, "dominant_GB/s": achieved, "dominant_frac": achieved / HBM_PEAK_GBS,
        "dominant_algorithmic_bytes": sbytes[dominant],
        "stages": stages, "ms_per_step_with_events": ms_per_step_ev,
        "ms_per_step_median_of_event_spans": ms_median_ev,
        "mfma_path_TFLOP/s": sum(sflops.values()) / (ms_per_step * 1e-3) / 1e12,
        "one_pass_K_bytes": total_bytes - sbytes["gram"],
        "workspace_MB": round(ws.numel() / 1e6, 1),
    }
    if not full:
        return res, (params, reqs, bufs, phi)

    # cold steps: the last-level cache (256 MB) is overwritten before each one
    if a.flush_cache:
        junk = torch.empty(512 << 20, dtype=torch.uint8, device=dev)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        acc = []
        for _ in range(steps):
            junk.fill_(1)
            e0.record()
            step(params)
            e1.record()
            torch.cuda.synchronize()
            acc.append(e0.elapsed_time(e1))
        res["cold_ms_per_step"] = sorted(acc)[len(acc) // 2]
        del junk

    # one step captured in a HIP graph and replayed (the call only launches kernels, so it can be)
    if a.graph:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step(params)
        for _ in range(warmup):
            graph.replay()
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        for _ in range(steps):
            graph.replay()
        torch.cuda.synchronize()
        res["graph_ms_per_step"] = (time.perf_counter() - t2) / steps * 1e3

    # the three unfused calls on the same buffers (scores then travel through HBM once more)
    scores = torch.empty(so[-1], dtype=torch.float32, device=dev)
    ev0 = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    acc = [0.0, 0.0, 0.0]
    for i in range(warmup + steps):
        ev0[0].record()
        C.compactor_score(params, reqs, scores=scores, status=bufs["status"], workspace=ws)
        ev0[1].record()
        C.compactor_select(params, reqs, scores, kept_idx=bufs["kept_idx"], kept_cnt=bufs["kept_cnt"],
                           workspace=ws)
        ev0[2].record()
        C.compactor_compact(params, reqs, bufs["kept_idx"], bufs["kept_cnt"], bufs["k_packed"],
                            bufs["v_packed"])
        ev0[3].record()
        torch.cuda.synchronize()
        if i >= warmup:
            for j in range(3):
                acc[j] += ev0[j].elapsed_time(ev0[j + 1]) / steps
    res["unfused_calls"] = {"score_ms": round(acc[0], 4), "select_ms": round(acc[1], 4),
                            "compact_ms": round(acc[2], 4), "total_ms": round(sum(acc), 4)}
    del scores
    return res, (params, reqs, bufs, phi)


# the other workloads of the benchmark set, reported beside the headline in "configs".  The order
# matters a little: where a workload's tensors land after the ones before it were freed moves its
# kernels by a few percent (config 3: 1.77 ms when it runs first, 1.85 to 1.89 ms after config 2
# or config 5, 1.80 ms in a process of its own).
OTHER_CONFIGS = [(3, False), (1, False), (2, False), (5, False), (5, True)]


def main():
    a = parse()
    if a.gpus != 1:
        print("bench.py measures one GPU: this library has no multi-GPU path (heads are independent, "
              "so more GPUs would each take a share of the heads with no communication). "
              "Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    import gc
    import torch
    from paper_2507_08143_amd import compactor as C
    from paper_2507_08143_amd import workloads as W

    dev = "cuda:0"
    torch.cuda.set_device(0)
    w = build_workload(W, a.config, dev, a.layers, a.exact)

    if a.attention or a.paged:
        res, (params, reqs, bufs, phi) = measure(a, torch, C, W, w, dev, full=False)
        (attention_mode if a.attention else paged_mode)(a, torch, C, W, w, reqs, params, bufs, dev)
        return

    copy_rates = None
    if a.calibrate_copy:
        src = torch.empty(1 << 28, dtype=torch.float32, device=dev).normal_()
        dst = torch.empty_like(src)
        torch.neg(src, out=dst)           # one elementwise kernel: reads 1 GiB, writes 1 GiB
        torch.cuda.synchronize()
        # the same two plain copies timed: what this GPU sustains on a dense read + write stream,
        # the pattern of the compaction stage without its indirection
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        copy_rates = {}
        for name, fn in (("torch_neg_GB/s", lambda: torch.neg(src, out=dst)),
                         ("torch_copy_GB/s", lambda: dst.copy_(src))):
            fn()
            e0.record()
            for _ in range(10):
                fn()
            e1.record()
            torch.cuda.synchronize()
            copy_rates[name] = round(10 * 2.0 * src.numel() * 4 / (e0.elapsed_time(e1) * 1e-3) / 1e9, 1)
        del src, dst

    res, (params, reqs, bufs, phi) = measure(a, torch, C, W, w, dev, full=True)
    dominant = res["dominant_kernel"]
    traffic = None
    if not a.layers and a.scope == "head" and not a.group_mb:
        traffic = MEASURED_TRAFFIC_BYTES.get((w.name, res["mode"].split()[0], dominant))

    out = {
        "metric": "tokens compressed/sec (score+select+compact) at 1 GPU",
        "value": res["value"], "unit": "tokens/s", "n_gpus": 1, "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": res["ms_per_step"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": w.name, "mode": res["mode"], "layers": w.layers, "kv_heads": w.kv_heads,
                   "head_dim": 128, "requests": res["requests"], "tokens": res["tokens"],
                   "head_rows": res["head_rows"], "kept_head_rows": res["kept_head_rows"],
                   "sketch_dim": w.sketch_dim, "group_mb": a.group_mb, "select_scope": a.scope,
                   "why": "largest single-GPU workload of the benchmark set" if a.config == 4 else "chosen with --config"},
        "roofline": {"bound": "hbm", "kernel": dominant, "achieved": res["dominant_GB/s"],
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": res["dominant_frac"],
                     "algorithmic_bytes": res["dominant_algorithmic_bytes"], "traffic": traffic},
        "path_hbm": {"algorithmic_bytes": res["algorithmic_bytes"],
                     "achieved_GB/s": res["algorithmic_bytes"] / (res["ms_per_step"] * 1e-3) / 1e9,
                     "frac_of_8TB/s": res["path_frac_of_8TB/s"],
                     # what a path whose second pass over K hit a cache would have to move
                     "one_pass_K_bytes": res["one_pass_K_bytes"]},
        "mfma": {"path_TFLOP/s": res["mfma_path_TFLOP/s"],
                 "frac_of_bf16_peak": res["mfma_path_TFLOP/s"] / MFMA_BF16_PEAK_TFLOPS},
        "stages": res["stages"], "ms_per_step_with_events": res["ms_per_step_with_events"],
        "ms_per_step_median_of_event_spans": res["ms_per_step_median_of_event_spans"],
        "unfused_calls": res["unfused_calls"],
    }
    for key in ("cold_ms_per_step", "graph_ms_per_step"):
        if key in res:
            out[key] = res[key]
    if copy_rates is not None:
        out["plain_copy_1GiB"] = copy_rates

    if not a.no_cpu_baseline:
        # the oracle on a bounded sample of the headline workload: all host cores, then one thread
        from oracle import compactor_oracle as O
        out["cpu_baseline"] = cpu_baseline(W, O, w, phi, a.cpu_seconds, a.cpu_threads)
        if a.cpu_threads == 0:
            out["cpu_baseline_1thread"] = cpu_baseline(W, O, w, phi, a.cpu_seconds, 1)

    # the other workloads of the set, each built, timed the same way and freed again
    if not a.only and not a.layers:
        del params, reqs, bufs, w
        gc.collect()
        torch.cuda.empty_cache()
        out["configs"] = []
        for cfg, exact in OTHER_CONFIGS:
            if cfg == a.config and exact == a.exact:
                continue
            wo = build_workload(W, cfg, dev, 0, exact)
            r, keep = measure(a, torch, C, W, wo, dev, full=False)
            out["configs"].append({
                "workload": r["workload"], "mode": r["mode"], "tokens": r["tokens"],
                "tokens_per_s": r["value"], "ms_per_step": round(r["ms_per_step"], 4),
                "path_frac_of_8TB/s": round(r["path_frac_of_8TB/s"], 4),
                "dominant_kernel": r["dominant_kernel"], "dominant_frac": round(r["dominant_frac"], 4),
                "stages_ms": {k_: v_["ms"] for k_, v_ in r["stages"].items()},
                "steps": r["steps"]})
            del wo, keep, r
            gc.collect()
            torch.cuda.empty_cache()
    print(json.dumps(out))


if __name__ == "__main__":
    main()
