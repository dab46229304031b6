#!/usr/bin/env python3
"""Denoising steps/s of the 1024-px DiT with classifier-free guidance on one MI355X.

One "step" is one complete model-function call (ServerlessT2I Sec. 4): the
stateless ``t2i_dit_step`` on 2 x 4096 image tokens (conditional + unconditional
branch) -- timestep embedding, every block's adaLN modulation, text projection
and cross K/V, patch embedding, 28 blocks (LN-mod, QKV, self-attention, gated
out-projection, cross-attention, MLP), final layer, guidance and the Euler
update -- on synthetic inputs already resident in HBM.

Prints ONE JSON line.  ``roofline`` is for the kernel with the largest share of
step time, timed with HIP events on the library's stream during the timed
steps; ``cpu_baseline`` is the oracle on the host cores on a bounded sample.

``--workload`` selects one of the other synthetic workloads instead (the
512-px DiT, the 3072-wide joint-attention model, the packed multi-request
batch) to report their achieved fractions the same way.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0          # MI355X HBM3E
WORKLOAD = "dit1024_cfg"

# HBM bytes per launch measured with rocprofv3 (FETCH_SIZE x 2.00 + WRITE_SIZE
# x 1.00, factors from a 1 GiB copy and a 1 GiB read through the direct-to-LDS
# load path),
# keyed by (workload, kernel class) with the source file it was measured on
# and the first 16 hex digits of the sha256 of that file's code (comments and
# blank lines removed, see code_digest): reported only while the code is
# unchanged.
MEASURED_TRAFFIC = {
    ("dit1024_cfg", "attn_self"): (107.1e6, "paper_2607_26566_amd/csrc/attention.hip", "05affee4fd72e1b5"),
}


def code_digest(path):
    """sha256 (16 hex digits) of a C++ source without // comments and blank
    lines, so that documentation edits leave a measurement valid."""
    import hashlib
    import re
    with open(path, encoding="utf-8") as f:
        lines = [re.sub(r"\s*//.*$", "", l).rstrip() for l in f]
    return hashlib.sha256("\n".join(l for l in lines if l).encode()).hexdigest()[:16]


def measured_traffic(workload, kernel):
    rec = MEASURED_TRAFFIC.get((workload, kernel))
    if rec is None:
        return None
    nbytes, src, digest = rec
    try:
        ok = code_digest(os.path.join(ROOT, src)) == digest
    except OSError:
        ok = False
    return nbytes if ok else None


def class_work(w):
    """Algorithmic work of each kernel class in ONE block at workload ``w``
    (FLOPs = 2MNK per GEMM and 4 Nq Nk d per attention head; bytes for the
    HBM-bound LN-mod: read fp32 x, write bf16 h), and its launches per block."""
    R = w.image_tokens * w.branches
    D, F = w.hidden, w.mlp_hidden
    seq = [w.tokens(r) for r in range(w.n_req)] * w.branches
    dh = w.heads * w.head_dim
    if w.arch == "mmdit":
        T = w.text_tokens
        Rt = R + len(seq) * T                       # text and image rows
        return {
            "gemm_qkv": ("flop", 2.0 * Rt * 3 * D * D, 2),
            "attn_self": ("flop", sum(4.0 * (n + T) ** 2 * dh for n in seq), 1),
            "gemm_o": ("flop", 2.0 * Rt * D * D, 2),
            "ln_mod": ("byte", 2 * Rt * D * (4.0 + 2.0), 4),
            "gemm_fc1": ("flop", 2.0 * Rt * F * D, 2),
            "gemm_fc2": ("flop", 2.0 * Rt * F * D, 2),
        }
    return {
        "gemm_qkv": ("flop", 2.0 * R * 3 * D * D, 1),
        "attn_self": ("flop", sum(4.0 * n * n * dh for n in seq), 1),
        "gemm_o": ("flop", 2.0 * R * D * D, 1),
        "gemm_xq": ("flop", 2.0 * R * D * D, 1),
        "attn_cross": ("flop", sum(4.0 * n * w.text_tokens * dh for n in seq), 1),
        "gemm_xo": ("flop", 2.0 * R * D * D, 1),
        "ln_mod": ("byte", 2 * R * D * (4.0 + 2.0), 2),
        "gemm_fc1": ("flop", 2.0 * R * F * D, 1),
        "gemm_fc2": ("flop", 2.0 * R * F * D, 1),
    }


def step_class_bytes(w):
    """Algorithmic HBM bytes of the once-per-step kernels: patch embedding
    (latent read, x0 and one residual copy per branch written), final layer
    (residual rows read; latent read, latent and velocity written) and the
    cache check (x0 and m_prev read, m written)."""
    T, D = w.image_tokens, w.hidden
    lat = 4.0 * T * w.patch_dim
    return {"embed": lat + 4.0 * T * D * (1 + w.branches),
            "final": 4.0 * T * D * w.branches + 3 * lat,
            "cache": 3 * 4.0 * T * D}


PEAK_F32_TFLOPS = 157.3        # MI355X fp32 vector (SIMT), 256 CU x 2.4 GHz


def step_flops(w):
    cw = class_work(w)
    return w.depth * sum(v for kind, v, _ in cw.values() if kind == "flop")


def cpu_baseline(w, W_host, min_seconds=10.0, max_passes=16):
    """The oracle on a bounded sample: block 0 of one step (every request and
    guidance branch), repeated until about ``min_seconds`` of CPU work have
    accumulated, the mean pass scaled to a whole step's blocks."""
    import numpy as np
    import synth
    from oracle import dit, mmdit
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count()
    wp = synth.reduced(w, depth=1)
    mm = w.arch == "mmdit"
    W = (mmdit if mm else dit).as_dict(wp, W_host)
    lats, texts = synth.latents(w), synth.texts(w)
    def one_pass():
        for r, lat in enumerate(lats):
            c = dit.conditioning(W, wp, 1.0)
            for txt in (texts[r], None)[:w.branches]:
                if mm:
                    xt, xi = mmdit.embed(W, wp, lat, txt)
                    mmdit.run_blocks(W, wp, xt, xi, c, lat.shape[1:], 0, 1)
                else:
                    y = dit.text_project(W, wp, txt if txt is not None
                                         else np.zeros((w.text_tokens, w.text_dim)))
                    dit.run_blocks(W, wp, dit.embed(W, wp, lat), y, c)

    t0 = time.perf_counter()
    passes = 0
    while passes < max_passes and (passes == 0 or time.perf_counter() - t0 < min_seconds):
        one_pass()
        passes += 1
    dt = time.perf_counter() - t0
    per_step = dt / passes * w.depth
    return {"value": round(1.0 / per_step, 6), "unit": "steps/s", "cores": int(cores),
            "kind": "oracle",
            "sample": f"float64 numpy oracle, block 0 of one {w.name} step for all "
                      f"{w.n_req} request(s) x {w.branches} guidance branch(es), {passes} "
                      f"pass(es) in {dt:.1f} s, mean pass scaled x{w.depth} to all blocks"}


def lora_cost(t2i, table, dev, rank):
    """Time merging one rank-``rank`` LoRA (alpha 1) into every 2-D weight of
    the blocks, as done once before sampling with an adapter: one batched
    launch per weight shape (t2i_op_lora_merge_batch), and for comparison one
    launch per weight (t2i_op_lora_merge)."""
    import torch
    idx = [i for i, (n, shp) in enumerate(table) if n.startswith("blocks.") and len(shp) == 2]
    g = torch.Generator(device="cuda").manual_seed(0)
    ad = {}
    for i in idx:
        n_out, n_in = table[i][1]
        key = (n_out, n_in)
        if key not in ad:
            ad[key] = (torch.randn(rank, n_in, generator=g, device="cuda").to(dev[i].dtype) * 0.01,
                       torch.randn(n_out, rank, generator=g, device="cuda").to(dev[i].dtype) * 0.01)
    by_shape = {}
    for i in idx:
        by_shape.setdefault(table[i][1], []).append(i)
    nbytes = sum(2 * dev[i].numel() * dev[i].element_size() +
                 sum(t.numel() * t.element_size() for t in ad[table[i][1]]) for i in idx)
    torch.cuda.synchronize()

    def timed(calls):
        evs = []
        for fn in calls:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            fn()
            e1.record()
            evs.append((e0, e1))
        torch.cuda.synchronize()
        return sum(e0.elapsed_time(e1) for e0, e1 in evs)

    batched = [lambda s=s, ix=ix: t2i.lora_merge_batch([dev[i] for i in ix], [ad[s][0]] * len(ix),
                                                       [ad[s][1]] * len(ix), 1.0)
               for s, ix in by_shape.items()]
    single = [lambda i=i: t2i.lora_merge(dev[i], ad[table[i][1]][0], ad[table[i][1]][1], 1.0)
              for i in idx]
    timed(batched)                       # warm-up
    ms = timed(batched)
    ms_single = timed(single)
    gbs = nbytes / (ms / 1e3) / 1e9
    return {"rank": rank, "layers": len(idx), "launches": sum((len(ix) + 63) // 64
                                                             for ix in by_shape.values()),
            "gpu_ms": round(ms, 3), "bytes": nbytes, "hbm_gbs": round(gbs, 1),
            "hbm_frac": round(gbs / PEAK_HBM_GBS, 4), "per_weight_launch_gpu_ms": round(ms_single, 3)}


def sched_bench(tenants=64, ready_per_tenant=4, decisions=20000):
    """Decisions per second of the vTime scheduler (submit + schedule +
    complete per decision) with `tenants` x `ready_per_tenant` ready
    invocations, on the host."""
    import numpy as np
    from paper_2607_26566_amd.scheduler import Scheduler

    def run(s, n):
        rng = np.random.default_rng(0)
        nid = 0
        for u in range(tenants):
            for _ in range(ready_per_tenant):
                s.submit(u, nid, float(rng.uniform(0.5, 10.0)), float(rng.uniform(0, 50)), 0.0)
                nid += 1
        t = 0.0
        t0 = time.perf_counter()
        for i in range(n):
            fn, u, est = s.schedule(t)
            s.complete(fn, est)
            t += est
            s.submit(u, nid, float(rng.uniform(0.5, 10.0)), float(rng.uniform(0, 50)), t)
            nid += 1
        return n / (time.perf_counter() - t0)

    rate = run(Scheduler(5.0), decisions)
    from oracle.sched import VTimeScheduler
    orate = run(VTimeScheduler(5.0), decisions // 20)
    return {"metric": "vTime scheduler decisions/s (host, via the Python binding)",
            "value": round(rate, 1), "unit": "decisions/s",
            "us_per_decision": round(1e6 / rate, 2),
            "config": {"tenants": tenants, "ready_invocations": tenants * ready_per_tenant},
            "cpu_baseline": {"value": round(orate, 1), "unit": "decisions/s", "cores": 1,
                             "kind": "oracle",
                             "sample": f"{decisions // 20} decisions of the Python oracle"}}


def request_flops(w, r):
    """GEMM + attention FLOPs of one request's rows in one step (all guidance
    branches), as class_work counts them."""
    n, D, F, M = w.tokens(r), w.hidden, w.mlp_hidden, w.text_tokens
    dh = w.heads * w.head_dim
    per_row = 2.0 * (3 * D * D + D * D + D * D + D * D + 2 * F * D)
    attn = 4.0 * n * n * dh + 4.0 * n * M * dh
    return w.depth * w.branches * (n * per_row + attn)


def cache_bench(t2i, m, w, x, x_init, hw, tx, sched, n_samples, warmup):
    """Whole samples with the step-skip cache on (tau of the workload, 0.1 if
    it has none): effective steps/s, and the FLOPs of the requests that ran
    their blocks (skipped requests cost x0 + R and the final layer only)."""
    import numpy as np
    import torch
    tau = w.cache_tau if w.cache_tau > 0 else 0.1
    toks = [w.tokens(r) for r in range(w.n_req)]
    state = m.new_cache_state(toks, w.branches)
    n = w.steps
    ts = np.array(sched)

    def one():
        x.copy_(x_init)
        return t2i.t2i_dit_sample(m, x, hw, tx, n, guidance=w.guidance, timesteps=ts,
                                  cache_tau=tau, cache_state=state)[0]
    from ctypes import c_double, c_int64, byref
    from paper_2607_26566_amd import _lib
    lib = t2i.load()
    for _ in range(warmup):
        one()
    torch.cuda.synchronize()
    logs = []
    # events around the cache-check kernels only (signal + decision, once per step)
    ci = _lib.KERNEL_CLASSES.index("cache")
    _lib.check(lib.t2i_dit_profile(m.h, 1 << ci), m.h)
    t0 = time.perf_counter()
    for _ in range(n_samples):
        logs.append(one())
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    tot, cnt = c_double(), c_int64()
    _lib.check(lib.t2i_dit_profile_read(m.h, ci, byref(tot), byref(cnt)), m.h)
    _lib.check(lib.t2i_dit_profile(m.h, 0), m.h)
    cache_bytes = step_class_bytes(w)["cache"] * cnt.value
    cache_gbs = cache_bytes / (tot.value / 1e3) / 1e9 if tot.value > 0 else 0.0
    rf = np.array([request_flops(w, r) for r in range(w.n_req)])
    executed = sum(float(((1 - lg) * rf[None, :]).sum()) for lg in logs)
    full = float(rf.sum()) * n * n_samples
    steps = n * n_samples
    skipped = int(sum(lg.sum() for lg in logs))
    return {
        "metric": f"effective denoising steps/s with the step-skip cache (tau {tau}) on {w.name}",
        "value": round(steps / el, 3), "unit": "steps/s", "steps": steps,
        "ms_per_step": round(el * 1e3 / steps, 3), "higher_is_better": True,
        "data": "synthetic", "cache_tau": tau,
        "skipped_request_steps": skipped, "request_steps": steps * w.n_req,
        "executed_flop_frac": round(executed / full, 4),
        "executed_tflops": round(executed / el / 1e12, 1),
        "executed_frac_of_peak": round(executed / el / 1e12 / PEAK_BF16_TFLOPS, 4),
        "hbm_frac": {"cache": {"gbs": round(cache_gbs, 1), "frac": round(cache_gbs / PEAK_HBM_GBS, 4),
                               "avg_launch_ms": round(tot.value / max(cnt.value, 1), 4)}},
        "skip_log_first_sample": logs[0].tolist(),
    }


PCIE5_X16_GBS = 63.0   # PCIe 5.0 x16, one direction: 32 GT/s x 16 lanes x 128/130


def loading_bench(t2i, m, cfg, w, dev, step, reps=3):
    """First-layers caching (Eq. 1-2) on this model: per-block copy time from
    pinned host memory, per-block compute time, and the end-to-end latency of
    one step started while the evicted blocks [L_e, L) are copied on a second
    stream, for every prefix L_e, next to Eq. 1 with the measured times."""
    import torch
    L = w.depth
    t0 = time.time()
    host = t2i.pack_blocks(cfg, dev)
    t2i.t2i_dit_host_tier(m, host)
    first, n, offs, bb = t2i.t2i_dit_block_layout(cfg)
    print(f"[bench] host tier packed: {L} x {bb / 1e6:.1f} MB in {time.time() - t0:.1f} s",
          file=sys.stderr, flush=True)
    comp = torch.cuda.current_stream()
    copy = torch.cuda.Stream()
    g = torch.randn(4096, 4096, device="cuda") * 1e-2

    def timed(fn):
        # a few ms of matmuls ahead of the timed region, so that every launch and
        # copy of it is queued before its first one can start
        a = g
        for _ in range(16):
            a = a @ g
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s.record(comp)
        fn()
        e.record(comp)
        torch.cuda.synchronize()
        return s.elapsed_time(e)

    def median(fn, before=None):
        xs = []
        for _ in range(reps):
            if before:
                before()
            xs.append(timed(fn))
        return sorted(xs)[len(xs) // 2]

    def load_on(stream):
        copy.wait_stream(comp)
        t2i.t2i_dit_load_async(m, stream)

    def load_only():
        load_on(copy)
        comp.wait_stream(copy)

    step()
    torch.cuda.synchronize()
    evict0 = lambda: t2i.t2i_dit_evict(m, 0)
    t_load_all = median(load_only, evict0)
    t_step = median(step)
    t_step0 = median(lambda: step(n_blocks=0))
    t_serial = median(lambda: (t2i.t2i_dit_load_async(m, comp), step()), evict0)
    tl, tc = t_load_all / L, (t_step - t_step0) / L
    e2e = []
    for le in range(L + 1):
        e2e.append(round(median(lambda: (load_on(copy), step()),
                                lambda: t2i.t2i_dit_evict(m, le)), 3))
        print(f"[bench] L_e={le}: {e2e[-1]:.2f} ms", file=sys.stderr, flush=True)
    t2i.t2i_dit_evict(m, L)
    eq1 = [round(t_step0 + max(L * tc, (L - le) * tl + tc), 3) for le in range(L + 1)]
    lp = t2i.t2i_first_layers(L, tl, tc)
    return {
        "metric": "first-layers caching: latency of one step that starts while blocks "
                  "[L_e, L) load from pinned host memory",
        "unit": "ms", "higher_is_better": False, "data": "synthetic",
        "config": {"workload": w.name, "blocks": L, "block_bytes": bb},
        "t_load_ms_per_block": round(tl, 4), "t_comp_ms_per_block": round(tc, 4),
        "t_rest_ms": round(t_step0, 3),
        "h2d_roofline": {"bound": "pcie", "achieved": round(bb * L / (t_load_all / 1e3) / 1e9, 1),
                         "peak": PCIE5_X16_GBS, "unit": "GB/s",
                         "frac": round(bb * L / (t_load_all / 1e3) / 1e9 / PCIE5_X16_GBS, 3)},
        "prefix_eq2": lp,
        "resident_ms": round(t_step, 3), "serial_ms": round(t_serial, 3),
        "ppl_0_ms": e2e[0], "ppl_prefix_ms": e2e[lp], "ppl_half_prefix_ms": e2e[lp // 2],
        "e2e_ms_by_prefix": e2e, "eq1_ms_by_prefix": eq1,
    }


WORKLOADS = {
    "dit1024_cfg": ("denoising steps/s at 1024px DiT; MFMA TFLOP/s as fraction of MI355X bf16 peak",
                    "dit1024_cfg: 1024px image, latent 4x128x128, patch 2 -> 4096 tokens x 2 "
                    "guidance branches (g=4.5), hidden 1152, 28 blocks, 16 heads x 72, MLP 4608, "
                    "120 text tokens x 4096, seed 2"),
    "dit512": ("denoising steps/s at 512px DiT (1024 tokens)",
               "dit512: 512px image, latent 4x64x64, patch 2 -> 1024 tokens, hidden 1152, "
               "28 blocks, 16 heads x 72, MLP 4608, 120 text tokens x 4096, seed 1"),
    "mmdit1024": ("denoising steps/s at 1024px joint-attention DiT (4096 image + 512 text tokens)",
                  "mmdit1024: latent 16x128x128, patch 2 -> 4096 image tokens + 512 text tokens "
                  "(4096 -> 3072), hidden 3072, 19 joint blocks, 24 heads x 128, MLP 12288, "
                  "2D RoPE, seed 3"),
    "tiny_f32": ("denoising steps/s of the tiny fp32 DiT (64 tokens)",
                 "tiny_f32: fp32, latent 4x16x16, patch 2 -> 64 tokens, hidden 128, 2 blocks, "
                 "2 heads x 64, MLP 512, 16 text tokens x 128, 4 steps, seed 0"),
    "packed8": ("denoising steps/s of a packed 8-request batch (12032 tokens)",
                "packed8: 3x256px + 3x512px + 2x1024px requests packed (256/1024/4096 tokens "
                "each, 12032 total), own timestep each, hidden 1152, 28 blocks, 16 heads x 72, "
                "cache skip off, seed 4"),
}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--workload", default=WORKLOAD, choices=sorted(WORKLOADS))
    ap.add_argument("--sched", action="store_true",
                    help="time only the vTime scheduler library (host CPU, no GPU)")
    ap.add_argument("--lora-rank", type=int, default=0,
                    help="also time merging a rank-R LoRA into every 2-D block weight")
    ap.add_argument("--loading", action="store_true",
                    help="time first-layers caching with progressive loading instead")
    ap.add_argument("--cache", action="store_true",
                    help="time whole samples with the step-skip cache on (effective steps/s)")
    ap.add_argument("--dma-calibration", action="store_true",
                    help="run only a 1 GiB read through the direct-to-LDS load path")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain 1 GiB device copy (HBM counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the denoising step "
              "is not sharded across GPUs in this build", file=sys.stderr)
        sys.exit(2)

    if args.sched:
        print(json.dumps(sched_bench()), flush=True)
        return

    import numpy as np
    import torch
    import synth
    import paper_2607_26566_amd as t2i
    from paper_2607_26566_amd import _lib

    if args.dma_calibration:
        import ctypes as C
        nbytes = 1 << 30
        a = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
        sink = torch.zeros(1024, dtype=torch.float32, device="cuda")
        lib = t2i.load()
        st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        for _ in range(5):
            _lib.check(lib.t2i_op_dma_read(C.c_void_p(a.data_ptr()), nbytes,
                                           C.c_void_p(sink.data_ptr()), st))
        torch.cuda.synchronize()
        print(json.dumps({"dma_bytes_read": nbytes, "launches": 5}))
        return

    if args.copy_calibration:
        n = 1 << 28                      # 2^28 floats = 1 GiB
        a = torch.ones(n, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        for _ in range(5):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": 4 * n, "copy_bytes_written": 4 * n, "launches": 5}))
        return

    w = synth.workload(args.workload)
    metric, desc = WORKLOADS[args.workload]
    cfg = t2i.Config.from_shape(w)
    table = t2i.weight_table(cfg)
    # weights generated and uploaded one tensor at a time (the 3072-wide model
    # has 6.5e9 parameters); the host keeps block 0 and the final layer for
    # the oracle baseline
    per_block = 16 if w.arch == "cross" else 20
    keep = set(range(8 + per_block)) | set(range(len(table) - 4, len(table)))
    dev, kept = [], {}
    t_w = time.time()
    for i in range(len(table)):
        a = synth.weights(w, table, pick=[i])[0]
        dev.append(t2i.upload([a], w.dtype)[0])
        if i in keep:
            kept[i] = a
        if time.time() - t_w > 20:
            print(f"[bench] weights {i + 1}/{len(table)}", file=sys.stderr, flush=True)
            t_w = time.time()
    W_host = [kept[i] for i in sorted(kept)]
    m = t2i.t2i_dit_init(cfg, dev)
    lats, texts = synth.latents(w), synth.texts(w)
    hw = list(w.requests)
    x = torch.from_numpy(np.concatenate([l.ravel() for l in lats])).cuda()
    tx = torch.from_numpy(np.stack(texts)).to("cuda", torch.bfloat16 if w.dtype == "bf16" else torch.float32)
    n = w.steps
    t0s = synth.start_times(w)
    sched = [[t0 * (1.0 - k / n) for t0 in t0s] for k in range(n + 1)]

    def run(i):
        k = i % n
        t2i.t2i_dit_step(m, x, hw, sched[k], tx, guidance=w.guidance, t_next=sched[k + 1])

    if args.loading:
        def one_step(n_blocks=-1):
            t2i.t2i_dit_step(m, x, hw, sched[0], tx, guidance=w.guidance, n_blocks=n_blocks)
        print(json.dumps(loading_bench(t2i, m, cfg, w, dev, one_step)), flush=True)
        return

    if args.cache:
        x_init = x.clone()
        out = cache_bench(t2i, m, w, x, x_init, hw, tx, sched, max(1, args.steps // n),
                          max(1, args.warmup // n + 1))
        # the same samples with the cache off, for comparison
        t_off = time.perf_counter()
        for _ in range(max(1, args.steps // n)):
            x.copy_(x_init)
            t2i.t2i_dit_sample(m, x, hw, tx, n, guidance=w.guidance, timesteps=np.array(sched))
        torch.cuda.synchronize()
        out["cache_off_steps_per_s"] = round(max(1, args.steps // n) * n / (time.perf_counter() - t_off), 3)
        out["config"] = {"workload": WORKLOADS[args.workload][1].replace("cache skip off", "cache skip on")}
        print(json.dumps(out), flush=True)
        return

    lib = t2i.load()
    # warmup; the last warmup pass times every kernel class to find the dominant one
    for i in range(max(args.warmup - 1, 0)):
        run(i)
    _lib.check(lib.t2i_dit_profile(m.h, (1 << len(_lib.KERNEL_CLASSES)) - 1), m.h)
    run(0)
    per_class = {}
    for ci, name in enumerate(_lib.KERNEL_CLASSES):
        tot, cnt = C_double(), C_int64()
        _lib.check(lib.t2i_dit_profile_read(m.h, ci, byref(tot), byref(cnt)), m.h)
        per_class[name] = (tot.value, cnt.value)
    dominant = max(per_class, key=lambda k: per_class[k][0])
    dom_idx = _lib.KERNEL_CLASSES.index(dominant)

    # timed region: events only around the dominant kernel class
    _lib.check(lib.t2i_dit_profile(m.h, 1 << dom_idx), m.h)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        run(i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    tot, cnt = C_double(), C_int64()
    _lib.check(lib.t2i_dit_profile_read(m.h, dom_idx, byref(tot), byref(cnt)), m.h)
    _lib.check(lib.t2i_dit_profile(m.h, 0), m.h)
    dom_avg_s = tot.value / 1e3 / max(cnt.value, 1)

    ms = elapsed * 1e3 / args.steps
    sps = args.steps / elapsed
    flops = step_flops(w)
    cw = class_work(w)
    # where the cross-attention runs inside its query projection (one kernel,
    # timed as gemm_xq), that kernel's work is both classes'
    xq_fused = ("attn_cross" in cw and per_class.get("attn_cross", (0, 0))[1] == 0
                and per_class.get("gemm_xq", (0, 0))[1] > 0)
    if xq_fused:
        cw["gemm_xq"] = ("flop", cw["gemm_xq"][1] + cw["attn_cross"][1], cw["gemm_xq"][2])
    kind, work_block, per_blk = cw[dominant]
    blocks = w.depth * args.steps                      # blocks executed in the timed region
    dom_s = tot.value / 1e3
    f32 = w.dtype != "bf16"
    peak_flops = PEAK_F32_TFLOPS if f32 else PEAK_BF16_TFLOPS
    if kind == "flop":
        ach = work_block * blocks / dom_s / 1e12
        roof = {"bound": "alu" if f32 else "mfma", "achieved": round(ach, 1), "peak": peak_flops,
                "unit": "TFLOP/s", "frac": round(ach / peak_flops, 4), "traffic": None}
    else:
        ach = work_block * blocks / dom_s / 1e9
        roof = {"bound": "hbm", "achieved": round(ach, 1), "peak": PEAK_HBM_GBS,
                "unit": "GB/s", "frac": round(ach / PEAK_HBM_GBS, 4), "traffic": None}
    roof["traffic"] = measured_traffic(args.workload, dominant)
    roof["kernel"] = dominant
    roof["avg_launch_ms"] = round(dom_avg_s * 1e3, 4)
    roof["launches"] = int(cnt.value)
    roof["work_per_launch"] = work_block / per_blk

    # per class: average launch time, and achieved rate over the profiled step
    kernel_ms = {k: round(v[0] / max(v[1], 1), 4) for k, v in per_class.items() if v[1]}
    class_rate = {}
    for k, (tms, c) in per_class.items():
        if not c or k not in cw:
            continue
        kd, wb, _ = cw[k]
        r = wb * w.depth / (tms / 1e3)
        class_rate[k] = (f"{r / 1e12:.1f} TFLOP/s" if kd == "flop" else f"{r / 1e9:.1f} GB/s")
    gemm_attn_ms = sum(v[0] for k, v in per_class.items() if k in cw and cw[k][0] == "flop")
    ln_ms = per_class["ln_mod"][0]
    ln_bytes = cw["ln_mod"][1] * w.depth
    # HBM fraction of the memory-bound kernels over the profiled step
    sb = step_class_bytes(w)
    hbm = {"ln_mod": (ln_bytes, ln_ms)}
    for k in ("embed", "final"):
        if per_class.get(k, (0, 0))[1]:
            hbm[k] = (sb[k], per_class[k][0])
    hbm_frac = {k: {"gbs": round(b / (t / 1e3) / 1e9, 1),
                    "frac": round(b / (t / 1e3) / 1e9 / PEAK_HBM_GBS, 4),
                    "avg_launch_ms": round(t / max(per_class[k][1], 1), 4)}
                for k, (b, t) in hbm.items() if t > 0}

    # a whole sample (conditioning and text computed once per sample)
    x.copy_(torch.from_numpy(np.concatenate([l.ravel() for l in lats])).cuda())
    torch.cuda.synchronize()
    ts = time.perf_counter()
    t2i.t2i_dit_sample(m, x, hw, tx, n, guidance=w.guidance, timesteps=np.array(sched))
    torch.cuda.synchronize()
    sample_s = time.perf_counter() - ts

    out = {
        "metric": metric,
        "value": round(sps, 3),
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16" if w.dtype == "bf16" else "f32",
        "data": "synthetic",
        "config": {"workload": desc, "global_batch": w.n_req * w.branches,
                   "seq_len": max(w.tokens(r) for r in range(w.n_req)),
                   "parallelism": "none (1 GPU)"},
        "roofline": roof,
        "gemm_attn_tflops_step": round(flops * sps / 1e12, 1),
        "gemm_attn_frac_of_peak_step": round(flops * sps / 1e12 / peak_flops, 4),
        "gemm_attn_tflops_kernels": round(flops / (gemm_attn_ms / 1e3) / 1e12, 1),
        "gemm_attn_frac_of_peak_kernels": round(flops / (gemm_attn_ms / 1e3) / 1e12 / peak_flops, 4),
        "ln_mod_gbs": round(ln_bytes / (ln_ms / 1e3) / 1e9, 1) if ln_ms > 0 else None,
        "hbm_frac": hbm_frac,
        "images_per_s": round(w.n_req / sample_s, 3),
        "sample_steps_per_s": round(n / sample_s, 3),
        "kernel_avg_ms": kernel_ms,
        "gemm_xq_includes_cross_attention": xq_fused,
        "kernel_class_rate": class_rate,
        "flops_per_step": flops,
    }
    if args.lora_rank:
        out["lora_merge"] = lora_cost(t2i, table, dev, args.lora_rank)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, W_host)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    from ctypes import c_double as C_double, c_int64 as C_int64, byref
    main()
