#!/usr/bin/env python3
"""Benchmark of the aLoRA hot path on one MI355X.

A step is one pass of the whole hot path (row preparation, fused base + gated low-rank QKV
projection, rotary embedding + cache append, attention over [base prefix ; adapted suffix])
over one batch of seeded synthetic input that is already resident in HBM.

    python bench.py [--workload c5|c2|c3|c4|c4x16|r2|r3|r3p] [--steps K] [--warmup W]

prints ONE JSON line: suffix tokens/s, ms per step, the roofline of the dominant kernel
(per-kernel durations from HIP events recorded by the library on the launch stream) and the
CPU oracle timed on the host cores on the same workload.  The default workload is c5, the
32-layer first-token pass at 32k context with its k = 0 full-LoRA recompute (the configuration
the metric is quoted on); its line also carries the c3 record (MFMA fractions of the projection
and prefill attention) and the c4 record (HBM fraction of decode attention) under "also".
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
PEAK_BF16_TFLOPS = 2516.6
MFMA_RIDGE = PEAK_BF16_TFLOPS * 1e12 / (PEAK_HBM_GBS * 1e9)      # flop per byte where the two rooflines meet


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=0)
    ap.add_argument("--warmup", type=int, default=0)
    ap.add_argument("--workload", default="c5", choices=["c2", "c3", "c4", "c4x16", "c4s", "c5", "c5n", "r2", "r3", "r3p", "copy"],
                    help="c5 (default): the first-token workload the metric is quoted on, with the c3 and c4 records "
                         "alongside; copy: a plain 1 GiB device copy, the known-size kernel that calibrates the HBM counters")
    ap.add_argument("--only", action="store_true", help="c5 only: leave out the c3 and c4 records")
    ap.add_argument("--rotate", type=int, default=-1,
                    help="distinct weight/cache sets cycled through so the last-level cache cannot hold the working set")
    ap.add_argument("--layers", type=int, default=0, help="c5 only: number of layers (default 32)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--variant", default="both", choices=["both", "shared", "private"],
                    help="r3 / r3p only: time the batch with shared context rows, with private copies, or both (default); "
                         "one variant per process is what a profiler run wants")
    ap.add_argument("--no-full-lora", action="store_true", help="c5 only: skip the k=0 recompute baseline")
    ap.add_argument("--plain", action="store_true", help="force the plain fp32-FMA kernels")
    ap.add_argument("--adapt-rest", action="store_true",
                    help="c5 only: adapters on W_o and the MLP linears too (Eq.6 on every linear of the layer)")
    ap.add_argument("--opt", action="append", default=[], help="library option key=value (repeatable)")
    return ap.parse_args()


# ------------------------------------------------------------------------------------------
# algorithmic work per kernel launch (what the method must do, never what a kernel happens to do)
# ------------------------------------------------------------------------------------------
def algorithmic_work(batch, shape, n_layers=1):
    esz = 2 if shape.dtype == "bf16" else 4
    T = batch.T
    d, N, r = shape.d, shape.n_qkv, shape.rank
    active_rows = sum(max(0, min(S, P + S - k)) if a >= 0 else 0
                      for P, S, k, a in zip(batch.P, batch.S, batch.k, batch.adapter))
    n_ad_used = len({a for a in batch.adapter if a >= 0})
    w = {}
    qkv_flops = 2.0 * T * d * N + 2.0 * active_rows * r * (3 * d + N)
    qkv_bytes = esz * (N * d + T * d + T * N + n_ad_used * r * (3 * d + N))
    w["qkv_gemm"] = dict(flops=qkv_flops, bytes=qkv_bytes)
    attn_flops = sum(4.0 * shape.head_dim * shape.n_q_heads * sum(range(P + 1, P + S + 1))
                     for P, S in zip(batch.P, batch.S))
    kv_bytes = sum((P + S) * 2 * shape.n_kv * esz for P, S in zip(batch.P, batch.S) if S > 0)
    w["attn_prefill"] = dict(flops=attn_flops, bytes=kv_bytes + 2 * T * shape.n_q * esz)
    w["attn_decode"] = dict(flops=attn_flops, bytes=kv_bytes)
    w["prep_rows"] = dict(flops=4.0 * T * d, bytes=2 * T * d * esz)
    w["rope_append"] = dict(flops=6.0 * T * (shape.n_q + shape.n_kv), bytes=T * N * esz * 2)
    w["attn_merge"] = dict(flops=0.0, bytes=T * shape.n_q * esz)
    if shape.intermediate:
        I = shape.intermediate
        w["o_proj"] = dict(flops=2.0 * T * d * shape.n_q, bytes=esz * (d * shape.n_q + T * shape.n_q + 2 * T * d))
        w["gate_up"] = dict(flops=4.0 * T * d * I, bytes=esz * (2 * I * d + T * d + 2 * T * I))
        w["down_proj"] = dict(flops=2.0 * T * d * I, bytes=esz * (I * d + T * I + 2 * T * d))
        w["mlp_norm"] = dict(flops=4.0 * T * d, bytes=2 * T * d * esz)
        w["silu_mul"] = dict(flops=4.0 * T * I, bytes=3 * T * I * esz)
    return w


# HBM traffic per launch (roofline.traffic): rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE per dispatch, calibrated on a
# plain copy of known size.  bench.py cannot read hardware counters itself; the figures come from
# profiles/traffic.json, which paper_2504_12397_amd/profile_summary.py writes from the counter runs of the kernels
# as committed (it records the kernel's symbol there).  A workload/kernel pair that is not in that file reports null.
def measured_traffic(workload, kernel):
    try:
        table = json.load(open(os.path.join(ROOT, "profiles", "traffic.json")))
    except (OSError, ValueError):
        return None
    rec = table.get(f"{workload}/{kernel}")
    return None if rec is None else float(rec["fetch_bytes"]) + float(rec["write_bytes"])


def roofline_of(kernel, work, avg_ms):
    flops, nbytes = work["flops"], work["bytes"]
    t_mfma = flops / (PEAK_BF16_TFLOPS * 1e12)
    t_hbm = nbytes / (PEAK_HBM_GBS * 1e9)
    sec = avg_ms * 1e-3
    if t_mfma >= t_hbm:
        ach = flops / sec / 1e12
        return dict(kernel=kernel, bound="mfma", achieved=ach, peak=PEAK_BF16_TFLOPS, unit="TFLOP/s",
                    frac=ach / PEAK_BF16_TFLOPS, traffic=None, avg_ms=avg_ms)
    ach = nbytes / sec / 1e9
    return dict(kernel=kernel, bound="hbm", achieved=ach, peak=PEAK_HBM_GBS, unit="GB/s", frac=ach / PEAK_HBM_GBS,
                traffic=None, avg_ms=avg_ms)


# ------------------------------------------------------------------------------------------
def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (run with --gpus 1)", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch
    from paper_2504_12397_amd import binding as ab, workloads as wl

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    torch.cuda.set_device(0)
    name = args.workload
    if name == "copy":
        n = 1 << 30
        src = torch.empty(n, dtype=torch.uint8, device=dev).random_()
        dst = torch.empty_like(src)
        steps = args.steps or 10
        for _ in range(2):
            dst.copy_(src)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            dst.copy_(src)
        torch.cuda.synchronize()
        sec = (time.perf_counter() - t0) / steps
        print(json.dumps({"metric": "device_copy", "bytes_read": n, "bytes_written": n, "steps": steps,
                          "ms_per_step": sec * 1e3, "GBps_read_plus_write": 2 * n / sec / 1e9}))
        return
    if name == "r2":
        return regime2(args, ab, wl, torch, np, dev)
    if name in ("r3", "r3p"):
        return regime3(args, ab, wl, torch, np, dev, prefill=name == "r3p")
    if name == "c5n":
        return evaluators(args, ab, wl, torch, np, dev)
    # (c4s carries no cpu_baseline: the oracle sample of c4 covers its attention block, the stack's other linears
    # are those of c5's sample)
    result = run_workload(name, args, ab, wl, torch, np, dev, cpu=not args.no_cpu_baseline and name != "c4s")
    if name == "c5" and not args.only:
        # The metric is quoted on c5 (first-token latency against the k = 0 recompute); its two roofline claims
        # live on other shapes -- the MFMA fraction of the projection and prefill attention on the mixed batch c3,
        # the HBM fraction of decode attention on c4 -- so the same line carries those records, each with its own
        # per-kernel rooflines, measured in this run.
        import copy
        sub = copy.copy(args)
        sub.steps = sub.warmup = 0
        sub.rotate = -1
        also = {}
        for extra in ("c3", "c4"):
            torch.cuda.empty_cache()
            also[extra] = run_workload(extra, sub, ab, wl, torch, np, dev, cpu=False)
        result["also"] = also
    print(json.dumps(result))


def run_workload(name, args, ab, wl, torch, np, dev, cpu=True):
    """One workload: timed steps, the same steps again with per-kernel HIP events, rooflines, and (cpu=True) the
    oracle on a bounded sample.  Returns the record."""
    # c4x16: 16 tokens per sequence of the c4 batch (the length of an evaluator's answer, Section 3) through one call of
    # alora_decode_steps, which has the inputs of all of them: its launches do the work of 16 new rows per sequence
    n_dec = 1
    if name == "c4x16":
        name, n_dec = "c4", 16
    # c4s: the c4 decode step through the whole stack (alora_stack_decode: attention, output projection and MLP of
    # every layer), what a token of the batch costs end to end
    stack_decode = name == "c4s"
    if stack_decode:
        name = "c4"
    batch = {"c2": wl.config2, "c3": wl.config3, "c4": wl.config4, "c5": wl.config5}[name]()
    shape = batch.shape
    n_layers = 1
    if stack_decode:
        import dataclasses
        shape = dataclasses.replace(shape, intermediate=wl.SHAPE_8B_STACK.intermediate)
        n_layers = args.layers or wl.N_LAYERS_STACK
    if name == "c5":
        n_layers = args.layers or wl.N_LAYERS_STACK
        if args.adapt_rest:
            import dataclasses
            shape = dataclasses.replace(shape, adapt_rest=True)
    steps = args.steps or (10 if stack_decode else {"c2": 200, "c3": 60, "c4": 50, "c5": 10}[name])
    warmup = args.warmup or (2 if stack_decode else {"c2": 20, "c3": 15, "c4": 5, "c5": 2}[name])
    rotate = args.rotate if args.rotate >= 0 else {"c2": 8, "c3": 2, "c4": 1, "c5": 1}[name]
    rotate = max(1, rotate)

    ctx = ab.Context(0)
    if args.plain:
        ctx.set_option("kernels", 1)
    for kv in args.opt:
        key, val = kv.split("=")
        ctx.set_option(key, int(val))
    rng = wl.Rng(batch.seed, dev)

    def make_set(tag):
        layers = [ab.Layer(wl.make_layer(shape, rng, f"{tag}.L{l}"), shape.n_q_heads, shape.n_kv_heads,
                           shape.head_dim, shape.rms_eps, shape.rope_theta, shape.intermediate)
                  for l in range(n_layers)]
        caps = [P + S * n_dec + (16 if name == "c5" else 0) for P, S in zip(batch.P, batch.S)]      # c5: room to generate
        caches = []
        for l in range(n_layers):
            c = ab.KVCache(caps, shape.n_kv_heads, shape.head_dim, shape.torch_dtype, dev)
            caches.append(c)
        return layers, caches

    sets = [make_set(f"set{i}") for i in range(rotate)]
    x_new = wl.make_hidden(rng, "x_new", batch.T, shape)
    x_steps = out_steps = None
    if n_dec > 1:
        x_steps = wl.make_hidden(rng, "x_steps", n_dec * batch.T, shape).view(n_dec, batch.T, shape.d)
        out_steps = torch.empty((n_dec, batch.T, shape.n_q), dtype=shape.torch_dtype, device=dev)

    # ---- prefix caches: what the base model stored earlier -------------------------------
    def fill_prefix(layers, caches, tag):
        if name == "c2":
            # the real flow: a base-model prefill (adapter -1) of the prefix creates the cache
            xp = wl.make_hidden(rng, f"{tag}.x_prefix", batch.P[0], shape)
            ab.alora_prefill(ctx, layers[0], caches[0], xp, [0, batch.P[0]], [0], [-1])
        elif stack_decode:
            # (tens of GB over the layers: filled in place by the device generator)
            for c in caches:
                c.k.normal_()
                c.v.normal_()
                c.seq_len[:] = np.asarray(batch.P, dtype=np.int32)
        else:
            # prefixes too long for a base pass inside a benchmark: N(0,1) keys/values, the
            # distribution the seeded weights and inputs produce
            for l, c in enumerate(caches):
                for b, P in enumerate(batch.P):
                    k, v = wl.make_random_kv(rng, f"{tag}.kv{l}.{b}", P, shape)
                    o = int(c.seq_offset[b])
                    c.k[o:o + P] = k
                    c.v[o:o + P] = v
                    c.seq_len[b] = P
        torch.cuda.synchronize()

    for i, (layers, caches) in enumerate(sets):
        fill_prefix(layers, caches, f"set{i}")

    out = torch.empty((batch.T, shape.d if (name == "c5" or stack_decode) else shape.n_q), dtype=shape.torch_dtype, device=dev)

    def step(i, b=batch, x=x_new, o=out):
        layers, caches = sets[i % rotate]
        for c in caches:
            c.seq_len[:] = np.asarray(b.P, dtype=np.int32)
        if n_dec > 1:
            ab.alora_decode_steps(ctx, layers[0], caches[0], x_steps, b.k, b.adapter, out_steps)
        elif stack_decode:
            ab.alora_stack_decode(ctx, layers, caches, x, b.k, b.adapter, o)
        elif name == "c4":
            ab.alora_decode(ctx, layers[0], caches[0], x, b.k, b.adapter, o)
        elif name == "c5":
            ab.alora_stack_prefill(ctx, layers, caches, x, b.cu_seqlens, b.k, b.adapter, o)
        else:
            ab.alora_prefill(ctx, layers[0], caches[0], x, b.cu_seqlens, b.k, b.adapter, o)

    for i in range(warmup):
        step(i)
    torch.cuda.synchronize()
    # what the host spends enqueueing a step (six steps: nothing in the library waits for the GPU that early)
    t0 = time.perf_counter()
    for i in range(min(6, steps)):
        step(i)
    host_ms_per_step = (time.perf_counter() - t0) / min(6, steps) * 1e3
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        step(i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / steps * 1e3
    tok_s = batch.T * n_dec / (elapsed / steps)

    # ---- per-kernel durations: the same steps again with the library's event brackets ----
    ctx.set_option("profile", 1)
    ctx.profile_reset()
    for i in range(steps):
        step(i)
    torch.cuda.synchronize()
    prof = ctx.profile_read()
    ctx.set_option("profile", 0)
    run = batch
    if n_dec > 1:
        import dataclasses
        run = dataclasses.replace(batch, S=[S * n_dec for S in batch.S])
    work = algorithmic_work(run, shape, n_layers)
    kernels = {}
    for kname, rec in prof.items():
        avg = rec["ms"] / rec["launches"]
        per_step = rec["ms"] / steps
        rl = roofline_of(kname, work[kname], avg) if kname in work else None
        kernels[kname] = dict(avg_ms=round(avg, 5), ms_per_step=round(per_step, 5), launches=rec["launches"],
                              bound=rl["bound"] if rl else None, frac=round(rl["frac"], 4) if rl else None,
                              achieved=round(rl["achieved"], 1) if rl else None, unit=rl["unit"] if rl else None)
    dominant = max(prof, key=lambda k_: prof[k_]["ms"])
    roof = roofline_of(dominant, work[dominant], prof[dominant]["ms"] / prof[dominant]["launches"])
    roof["traffic"] = None if args.plain else measured_traffic(name, dominant)
    roof["algorithmic_bytes"] = work[dominant]["bytes"]
    roof["algorithmic_flops"] = work[dominant]["flops"]

    result = {
        "metric": "alora_suffix_prefill_tok_per_s" if name != "c4" else "alora_decode_tok_per_s",
        "value": tok_s, "unit": "tok/s", "n_gpus": 1, "steps": steps, "warmup": warmup,
        "ms_per_step": ms_per_step, "host_ms_per_step": round(host_ms_per_step, 4), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": shape.dtype, "data": "synthetic",
        "config": {"workload": "", "sequences": batch.n_seqs, "suffix_tokens": batch.T,
                   "prefix_tokens": int(sum(batch.P)), "rank": shape.rank, "layers": n_layers,
                   "rotating_buffer_sets": rotate, "kernels": "plain" if args.plain else "auto",
                   "adapted_linears": "q,k,v,o,gate,up,down" if getattr(shape, "adapt_rest", False) else "q,k,v"},
        "ttft_ms": ms_per_step,
        "roofline": roof,
        "kernels": kernels,
    }
    result["config"]["workload"] = {
        "c2": "c2: one 8B-class layer, bf16, 4096 cached base tokens + 256 adapted suffix tokens, rank 32",
        "c3": "c3: mixed batch, 16 sequences, prefix 512-8192, suffix 32-512, 4 rank-32 adapters, 3 base-only",
        "c4": "c4: decode step, 64 sequences x (16384 base + 64 adapted cached tokens), 1 new token each",
        "c5": "c5: %d-layer 8B-class stack, 32768 cached base tokens + 128 adapted suffix tokens, rank 64, "
              "time to the first adapter token against the k = 0 full-LoRA recompute" % n_layers,
    }[name]
    if stack_decode:
        result["config"]["workload"] = ("c4s: decode step through %d layers of the 8B-class stack (attention, output "
                                        "projection, SwiGLU MLP), 64 sequences x (16384 base + 64 adapted cached tokens)"
                                        % n_layers)
    if n_dec > 1:
        result["config"]["workload"] = ("c4x16: %d decode steps of the c4 batch, inputs at hand, in one call "
                                        "(64 sequences x 16448 cached tokens at the start)" % n_dec)
        result["config"]["decode_steps"] = n_dec
    if name != "c5":
        del result["ttft_ms"]

    # ---- full-LoRA baseline for the first-token workload: same kernels, k = 0, empty cache ----
    if name == "c5" and not args.no_full_lora:
        fb = wl.config5(full_lora=True)
        x_full = wl.make_hidden(rng, "x_full", fb.T, shape)
        out_full = torch.empty((fb.T, shape.d), dtype=shape.torch_dtype, device=dev)
        layers, caches = sets[0]

        def full_step():
            for c in caches:
                c.seq_len[:] = 0
            ab.alora_stack_prefill(ctx, layers, caches, x_full, fb.cu_seqlens, fb.k, fb.adapter, out_full)

        full_step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        n_full = 2
        for _ in range(n_full):
            full_step()
        torch.cuda.synchronize()
        full_ms = (time.perf_counter() - t0) / n_full * 1e3
        result["full_lora_ttft_ms"] = full_ms
        result["ttft_speedup_vs_full_lora"] = full_ms / ms_per_step
        # the recompute's own per-kernel times and rooflines (one more pass with the event brackets)
        ctx.set_option("profile", 1)
        ctx.profile_reset()
        full_step()
        torch.cuda.synchronize()
        fprof = ctx.profile_read()
        ctx.set_option("profile", 0)
        fwork = algorithmic_work(fb, shape, n_layers)
        fk = {}
        for kname, rec in fprof.items():
            avg = rec["ms"] / rec["launches"]
            rl = roofline_of(kname, fwork[kname], avg) if kname in fwork else None
            fk[kname] = dict(avg_ms=round(avg, 4), launches=rec["launches"], bound=rl["bound"] if rl else None,
                             frac=round(rl["frac"], 4) if rl else None)
        result["full_lora_kernels"] = fk
        del x_full, out_full

    # ---- first token id: final norm + vocabulary projection + greedy choice on the last row -----
    if name == "c5":
        V = 128256
        Wv = rng.normal("lm_head.W", (V, shape.d), 1.0 / np.sqrt(shape.d), dtype=shape.torch_dtype)
        gf = rng.normal("lm_head.gain", (shape.d,), 0.1, 1.0, dtype=shape.torch_dtype)
        last = out[-1:].contiguous()
        for _ in range(3):
            ab.alora_lm_head(ctx, last, gf, shape.rms_eps, Wv)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(20):
            ab.alora_lm_head(ctx, last, gf, shape.rms_eps, Wv)
        torch.cuda.synchronize()
        head_ms = (time.perf_counter() - t0) / 20 * 1e3
        result["lm_head_ms"] = head_ms
        result["lm_head_GBps"] = V * shape.d * 2 / (head_ms * 1e-3) / 1e9
        result["ttft_to_token_id_ms"] = ms_per_step + head_ms
        # ---- the rest of a 16-token evaluator generation (Section 3: every adapter call generates 16 tokens): 15
        # decode steps through the stack, each followed by the output head.  A random hidden row stands in for the
        # embedding of the token just generated.
        layers, caches = sets[0]
        x_tok = wl.make_hidden(rng, "x_tok", batch.n_seqs, shape)
        out_tok = torch.empty((batch.n_seqs, shape.d), dtype=shape.torch_dtype, device=dev)
        after_prefill = np.asarray([P + S for P, S in zip(batch.P, batch.S)], dtype=np.int32)

        def generate(n):
            for c in caches:
                c.seq_len[:] = after_prefill
            for _ in range(n):
                ab.alora_stack_decode(ctx, layers, caches, x_tok, batch.k, batch.adapter, out_tok)
                ab.alora_lm_head(ctx, out_tok, gf, shape.rms_eps, Wv)

        generate(3)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        generate(15)
        torch.cuda.synchronize()
        dec_ms = (time.perf_counter() - t0) / 15 * 1e3
        result["decode_step_ms"] = dec_ms
        result["evaluator_16_tokens_ms"] = ms_per_step + head_ms + 15 * dec_ms
        if "full_lora_ttft_ms" in result:
            # a LoRA evaluator's decode steps are the same calls over the same number of cached rows
            result["full_lora_evaluator_16_tokens_ms"] = result["full_lora_ttft_ms"] + head_ms + 15 * dec_ms
            result["evaluator_speedup_vs_full_lora"] = (result["full_lora_evaluator_16_tokens_ms"] /
                                                        result["evaluator_16_tokens_ms"])
        for c in caches:
            c.seq_len[:] = np.asarray(batch.P, dtype=np.int32)
        del Wv

    # ---- the CPU oracle on the same workload, timed on the host cores -------------------------
    if cpu:
        result["cpu_baseline"] = cpu_baseline(name, batch, shape, sets[0], x_new, n_layers)
    ctx.close()
    del sets, out, x_new
    torch.cuda.empty_cache()
    return result


def regime2(args, ab, wl, torch, np, dev):
    """Section 2 ("Cache reuse patterns"), second regime: the adapter call prefills uncached context with base weights up to k
    and the next base-model turn reuses those rows; compared with the base model prefilling the
    context again (what it costs when the adapter call's cache cannot be reused)."""
    first, then = wl.regime2()
    shape = first.shape
    steps, warmup = args.steps or 20, args.warmup or 3
    ctx = ab.Context(0)
    for kv in args.opt:
        key, val = kv.split("=")
        ctx.set_option(key, int(val))
    rng = wl.Rng(first.seed, dev)
    layer = ab.Layer(wl.make_layer(shape, rng, "r2.L0"), shape.n_q_heads, shape.n_kv_heads, shape.head_dim,
                     shape.rms_eps, shape.rope_theta, shape.intermediate)
    cache = ab.KVCache([first.T + then.T], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, dev)
    x1 = wl.make_hidden(rng, "r2.x1", first.T, shape)
    x2 = wl.make_hidden(rng, "r2.x2", then.T, shape)
    o1 = torch.empty((first.T, shape.n_q), dtype=shape.torch_dtype, device=dev)
    o2 = torch.empty((then.T, shape.n_q), dtype=shape.torch_dtype, device=dev)
    x_re = torch.cat([x1[:then.P[0]], x2]).contiguous()
    o_re = torch.empty((x_re.shape[0], shape.n_q), dtype=shape.torch_dtype, device=dev)

    def step(_):
        cache.seq_len[0] = 0
        ab.alora_prefill(ctx, layer, cache, x1, first.cu_seqlens, first.k, first.adapter, o1)
        cache.seq_len[0] = then.P[0]            # drop the adapted rows, keep the base rows before k
        ab.alora_prefill(ctx, layer, cache, x2, then.cu_seqlens, then.k, then.adapter, o2)

    def reprefill(_):
        cache.seq_len[0] = 0
        ab.alora_prefill(ctx, layer, cache, x_re, [0, x_re.shape[0]], [0], [-1], o_re)

    def timed(f, n):
        for i in range(warmup):
            f(i)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(n):
            f(i)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / n

    sec = timed(step, steps)
    ctx.set_option("profile", 1)
    ctx.profile_reset()
    cache.seq_len[0] = then.P[0]
    for _ in range(steps):
        ab.alora_prefill(ctx, layer, cache, x2, then.cu_seqlens, then.k, then.adapter, o2)
        cache.seq_len[0] = then.P[0]
    torch.cuda.synchronize()
    turn_prof = ctx.profile_read()
    ctx.profile_reset()
    for i in range(steps):
        step(i)
    torch.cuda.synchronize()
    prof = ctx.profile_read()
    ctx.set_option("profile", 0)
    turn_ms = sum(r["ms"] for r in turn_prof.values()) / steps
    sec_re = timed(reprefill, max(2, steps // 2))
    w1, w2 = algorithmic_work(first, shape), algorithmic_work(then, shape)
    dominant = max(prof, key=lambda k_: prof[k_]["ms"])
    both = {q: (w1[dominant][q] + w2[dominant][q]) / 2 for q in ("flops", "bytes")}     # per launch, two per step
    roof = roofline_of(dominant, both, prof[dominant]["ms"] / prof[dominant]["launches"])
    result = {
        "metric": "alora_suffix_prefill_tok_per_s", "value": (first.T + then.T) / sec, "unit": "tok/s", "n_gpus": 1,
        "steps": steps, "warmup": warmup, "ms_per_step": sec * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": shape.dtype, "data": "synthetic",
        "config": {"workload": "r2: adapter call over 4096 uncached context tokens + 256 adapted tokens (k=4096, P=0), "
                               "then a 256-token base-model turn on the 4096 base rows that call created",
                   "rank": shape.rank, "layers": 1},
        "roofline": roof,
        "kernels": {k_: dict(avg_ms=round(r["ms"] / r["launches"], 5), launches=r["launches"]) for k_, r in prof.items()},
        "base_turn_with_reuse_ms": turn_ms,
        "base_turn_reprefilling_context_ms": sec_re * 1e3,
        "base_turn_saving": sec_re * 1e3 / turn_ms,
    }
    print(json.dumps(result))
    ctx.close()


def regime3(args, ab, wl, torch, np, dev, prefill=False):
    """Section 2 ("Cache reuse patterns"), third regime: sequences that run different adapters over the same context
    read one physical copy of its cache rows, and their rows share workgroups for that part (a decode step packs
    four sequences to a workgroup; a prefill of invocation sequences packs the rows of neighbouring sequences up
    to a full query tile); compared with the same batch holding a private copy of the context per sequence."""
    batch, ctx_of, C0 = wl.regime3_prefill() if prefill else wl.regime3()
    shape = batch.shape
    n = batch.n_seqs
    n_ctx = max(ctx_of) + 1
    own = batch.P[0] - C0
    S = batch.S[0]
    kname = "attn_prefill" if prefill else "attn_decode"
    steps, warmup = args.steps or 30, args.warmup or 5
    ctx = ab.Context(0)
    for kv in args.opt:
        key, val = kv.split("=")
        ctx.set_option(key, int(val))
    rng = wl.Rng(batch.seed, dev)
    layer = ab.Layer(wl.make_layer(shape, rng, "r3.L0"), shape.n_q_heads, shape.n_kv_heads, shape.head_dim,
                     shape.rms_eps, shape.rope_theta, shape.intermediate)
    x = wl.make_hidden(rng, "r3.x", n * S, shape)
    out = torch.empty((n * S, shape.n_q), dtype=shape.torch_dtype, device=dev)
    cu = [b * S for b in range(n + 1)]

    def make_cache(shared):
        caps = [(own if shared else batch.P[b]) + S for b in range(n)] + ([C0] * n_ctx if shared else [])
        c = ab.KVCache(caps, shape.n_kv_heads, shape.head_dim, shape.torch_dtype, dev)
        c.k.normal_()
        c.v.normal_()
        for b in range(n):
            c.seq_len[b] = batch.P[b]
            if shared:
                c.share_prefix(b, int(c.seq_offset[n + ctx_of[b]]), C0)
        return c

    def run(shared):
        c = make_cache(shared)

        def step():
            c.seq_len[:n] = np.asarray(batch.P, dtype=np.int32)
            if prefill:
                ab.alora_prefill(ctx, layer, c, x, cu, batch.k, batch.adapter, out)
            else:
                ab.alora_decode(ctx, layer, c, x, batch.k, batch.adapter, out)

        for _ in range(warmup):
            step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            step()
        torch.cuda.synchronize()
        sec = (time.perf_counter() - t0) / steps
        ctx.set_option("profile", 1)
        ctx.profile_reset()
        for _ in range(steps):
            step()
        torch.cuda.synchronize()
        prof = ctx.profile_read()
        ctx.set_option("profile", 0)
        del c
        return sec, prof

    if args.variant == "private":
        sec, prof = run(False)
        sec_private, prof_private = sec, prof
    else:
        sec, prof = run(True)
        sec_private, prof_private = run(False) if args.variant == "both" else (None, None)

    esz = 2
    avg = prof[kname]["ms"] / prof[kname]["launches"]
    avg_private = prof_private[kname]["ms"] / prof_private[kname]["launches"] if prof_private else None
    # the rows that exist: every context once (or once per sequence when each holds a private copy) + the own rows
    alg_bytes = ((n if args.variant == "private" else n_ctx) * C0 + n * (own + S)) * 2 * shape.n_kv * esz
    if prefill:
        # causal attention of S new tokens over P cached ones: 4 * head_dim flops per (query head, visible key)
        alg = n * 4 * shape.head_dim * shape.n_q_heads * (S * batch.P[0] + S * (S + 1) // 2)
        roof = dict(kernel=kname, bound="mfma", achieved=alg / (avg * 1e-3) / 1e12, peak=PEAK_BF16_TFLOPS,
                    unit="TFLOP/s", frac=alg / (avg * 1e-3) / 1e12 / PEAK_BF16_TFLOPS,
                    traffic=measured_traffic("r3pp" if args.variant == "private" else "r3p", kname), avg_ms=avg, algorithmic_flops=alg,
                    algorithmic_bytes=alg_bytes, hbm_frac=alg_bytes / (avg * 1e-3) / 1e9 / PEAK_HBM_GBS)
        what = ("r3p: prefill of %d invocation sequences of %d tokens = %d contexts of %d cached base tokens x %d adapter "
                "calls, the context rows stored once per context" % (n, S, n_ctx, C0, n // n_ctx))
    else:
        roof = dict(kernel=kname, bound="hbm", achieved=alg_bytes / (avg * 1e-3) / 1e9, peak=PEAK_HBM_GBS, unit="GB/s",
                    frac=alg_bytes / (avg * 1e-3) / 1e9 / PEAK_HBM_GBS, traffic=None, avg_ms=avg,
                    algorithmic_bytes=alg_bytes)
        what = ("r3: decode step, %d sequences = %d contexts of %d cached base tokens x %d adapters, %d own "
                "adapted rows each, the context rows stored once per context" % (n, n_ctx, C0, n // n_ctx, own))
    result = {
        "metric": "alora_suffix_prefill_tok_per_s" if prefill else "alora_decode_tok_per_s", "value": n * S / sec,
        "unit": "tok/s", "n_gpus": 1, "steps": steps, "warmup": warmup,
        "ms_per_step": sec * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": shape.dtype,
        "data": "synthetic",
        "config": {"workload": what, "rank": shape.rank, "layers": 1},
        "roofline": roof,
        "kernels": {k_: dict(avg_ms=round(r["ms"] / r["launches"], 5), launches=r["launches"]) for k_, r in prof.items()},
        "variant": args.variant,
    }
    if args.variant == "both":
        result.update({"private_copies_ms_per_step": sec_private * 1e3, "private_copies_%s_ms" % kname: avg_private,
                       "speedup_vs_private_copies": sec_private / sec,
                       "%s_speedup_vs_private_copies" % kname: avg_private / avg})
    if args.variant == "private":
        result["config"]["workload"] = result["config"]["workload"].replace(
            "the context rows stored once per context", "every sequence holding a private copy of its context's rows")
    print(json.dumps(result))
    ctx.close()


def evaluators(args, ab, wl, torch, np, dev):
    """Config 5 with N evaluators on one context, through the whole stack (Proposition 2 for N adapters; Section 2,
    "Cache reuse patterns", third regime; Section 3's 16-token evaluator answers): one alora_stack_prefill over the N
    invocation sequences, which all name the single copy of the context's rows, then 15 x (alora_stack_decode +
    alora_lm_head) for the N sequences; beside it the same calls with a private copy of the context per sequence
    and the call for a single evaluator."""
    batch = wl.evaluators_on_one_context()
    shape = batch.shape
    n, C0, S = batch.n_seqs, batch.P[0], batch.S[0]
    n_layers = args.layers or wl.N_LAYERS_STACK
    n_gen = 16
    steps, warmup = args.steps or 8, args.warmup or 2
    ctx = ab.Context(0)
    for kv in args.opt:
        key, val = kv.split("=")
        ctx.set_option(key, int(val))
    rng = wl.Rng(batch.seed, dev)
    layers = [ab.Layer(wl.make_layer(shape, rng, f"c5n.L{l}"), shape.n_q_heads, shape.n_kv_heads, shape.head_dim,
                       shape.rms_eps, shape.rope_theta, shape.intermediate) for l in range(n_layers)]
    x = wl.make_hidden(rng, "c5n.x", n * S, shape)
    x_tok = wl.make_hidden(rng, "c5n.x_tok", n, shape)
    out = torch.empty((n * S, shape.d), dtype=shape.torch_dtype, device=dev)
    out_tok = torch.empty((n, shape.d), dtype=shape.torch_dtype, device=dev)
    V = 128256
    Wv = rng.normal("lm_head.W", (V, shape.d), 1.0 / np.sqrt(shape.d), dtype=shape.torch_dtype)
    gf = rng.normal("lm_head.gain", (shape.d,), 0.1, 1.0, dtype=shape.torch_dtype)

    def make_caches(shared, m):
        caches = []
        for l in range(n_layers):
            caps = [(0 if shared else C0) + S + n_gen for _ in range(m)] + ([C0] if shared else [])
            c = ab.KVCache(caps, shape.n_kv_heads, shape.head_dim, shape.torch_dtype, dev)
            c.k.normal_()
            c.v.normal_()
            for b in range(m):
                c.seq_len[b] = C0
                if shared:
                    c.share_prefix(b, int(c.seq_offset[m]), C0)
            caches.append(c)
        return caches

    def run(shared, m, profile=False):
        caches = make_caches(shared, m)
        cu = [b * S for b in range(m + 1)]
        kk, ad = batch.k[:m], batch.adapter[:m]

        def first_tokens():
            for c in caches:
                c.seq_len[:m] = C0
            ab.alora_stack_prefill(ctx, layers, caches, x[:m * S], cu, kk, ad, out[:m * S])
            # the last row of every sequence goes through the output head
            last = out[:m * S].view(m, S, shape.d)[:, -1].contiguous()
            ab.alora_lm_head(ctx, last, gf, shape.rms_eps, Wv)

        def generate(k_steps):
            for _ in range(k_steps):
                ab.alora_stack_decode(ctx, layers, caches, x_tok[:m], kk, ad, out_tok[:m])
                ab.alora_lm_head(ctx, out_tok[:m], gf, shape.rms_eps, Wv)

        for _ in range(warmup):
            first_tokens()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            first_tokens()
        torch.cuda.synchronize()
        ttft = (time.perf_counter() - t0) / steps
        generate(2)
        torch.cuda.synchronize()
        for c in caches:
            c.seq_len[:m] = C0 + S
        t0 = time.perf_counter()
        generate(n_gen - 1)
        torch.cuda.synchronize()
        dec = (time.perf_counter() - t0) / (n_gen - 1)
        prof = None
        if profile:
            ctx.set_option("profile", 1)
            ctx.profile_reset()
            first_tokens()
            torch.cuda.synchronize()
            prof = ctx.profile_read()
            ctx.set_option("profile", 0)
        del caches
        torch.cuda.empty_cache()
        return ttft, dec, prof

    ttft, dec, prof = run(True, n, profile=True)
    ttft_private, dec_private, _ = run(False, n) if args.variant == "both" else (None, None, None)
    ttft_one, dec_one, _ = run(True, 1)
    avg = prof["attn_prefill"]["ms"] / prof["attn_prefill"]["launches"]
    alg = n * 4 * shape.head_dim * shape.n_q_heads * (S * C0 + S * (S + 1) // 2)
    alg_bytes = (C0 + n * S) * 2 * shape.n_kv * 2
    result = {
        "metric": "alora_suffix_prefill_tok_per_s", "value": n * S / ttft, "unit": "tok/s", "n_gpus": 1, "steps": steps,
        "warmup": warmup, "ms_per_step": ttft * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": shape.dtype, "data": "synthetic",
        "config": {"workload": "c5n: %d evaluators (one adapter each) x %d adapted tokens on one context of %d cached base "
                               "tokens stored once, %d layers, output head included" % (n, S, C0, n_layers),
                   "rank": shape.rank, "layers": n_layers},
        "roofline": dict(kernel="attn_prefill", bound="mfma", achieved=alg / (avg * 1e-3) / 1e12, peak=PEAK_BF16_TFLOPS,
                         unit="TFLOP/s", frac=alg / (avg * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, traffic=None, avg_ms=avg,
                         algorithmic_flops=alg, algorithmic_bytes=alg_bytes),
        "kernels": {k_: dict(avg_ms=round(r["ms"] / r["launches"], 5), launches=r["launches"]) for k_, r in prof.items()},
        "first_tokens_ms": ttft * 1e3, "first_tokens_ms_per_evaluator": ttft * 1e3 / n,
        "decode_step_ms": dec * 1e3, "evaluators_16_tokens_ms": (ttft + (n_gen - 1) * dec) * 1e3,
        "one_evaluator_first_token_ms": ttft_one * 1e3, "one_evaluator_decode_step_ms": dec_one * 1e3,
        "one_evaluator_16_tokens_ms": (ttft_one + (n_gen - 1) * dec_one) * 1e3,
        "speedup_vs_one_evaluator_at_a_time": n * (ttft_one + (n_gen - 1) * dec_one) / (ttft + (n_gen - 1) * dec),
    }
    if ttft_private is not None:
        result.update({"private_copies_first_tokens_ms": ttft_private * 1e3, "private_copies_decode_step_ms": dec_private * 1e3,
                       "private_copies_16_tokens_ms": (ttft_private + (n_gen - 1) * dec_private) * 1e3,
                       "speedup_vs_private_copies": (ttft_private + (n_gen - 1) * dec_private) / (ttft + (n_gen - 1) * dec)})
    print(json.dumps(result))
    ctx.close()


def cpu_baseline(name, batch, shape, first_set, x_new, n_layers):
    """The oracle as it stands, on a bounded sample of the workload (stated in "sample")."""
    import numpy as np
    import torch
    from oracle import alora_oracle as orc
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
    except Exception:
        cores = os.cpu_count() or 1
    layers, caches = first_set

    def host_layer(l):
        t = {k_: (v.cpu() if isinstance(v, torch.Tensor) else v) for k_, v in layers[l].t.items()}
        return orc.layer_from_tensors(t, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rms_eps,
                                      shape.rope_theta)

    # bounded sample: whole c2; 2 sequences of c3; 4 sequences of c4; one layer of c5
    seqs = {"c2": [0], "c3": [0, 1], "c4": [0, 1, 2, 3], "c5": [0]}[name]
    L0 = host_layer(0)
    xs = x_new.cpu().double().numpy()
    cu = batch.cu_seqlens
    data = []
    for b in seqs:
        o = int(caches[0].seq_offset[b])
        K = caches[0].k[o:o + batch.P[b]].cpu().double().numpy().reshape(batch.P[b], -1)
        V = caches[0].v[o:o + batch.P[b]].cpu().double().numpy().reshape(batch.P[b], -1)
        data.append((b, K, V, xs[cu[b]:cu[b + 1]]))
    if name == "c5":
        t = {k_: (v.cpu() if isinstance(v, torch.Tensor) else v) for k_, v in layers[0].t.items()}
        L0 = orc.layer_from_tensors(t, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rms_eps,
                                    shape.rope_theta)
    # repeat the sample until about 10 s of CPU work have been timed (at least once, at most 30 s)
    t0 = time.perf_counter()
    toks, reps = 0, 0
    while True:
        for b, K, V, x in data:
            o, kn, vn = orc.ref_cached(L0, K, V, batch.P[b], x, batch.k[b], batch.adapter[b], shape.dtype)
            if name == "c5":
                orc.layer_tail(L0, x, o, shape.dtype)
            toks += x.shape[0]
        reps += 1
        sec = time.perf_counter() - t0
        if sec >= 10.0 or (sec / reps) * (reps + 1) > 30.0:
            break
    scale_layers = n_layers if name == "c5" else 1
    return {"value": toks / (sec * scale_layers), "unit": "tok/s", "cores": int(cores), "kind": "oracle",
            "implementation": "float64 numpy (matrix products through the BLAS numpy links, multi-threaded); "
                              + ("one layer timed, scaled by the layer count (extrapolated)" if name == "c5" else "as timed"),
            "seconds": sec, "repetitions": reps,
            "sample": {"c2": "the whole workload (256 suffix tokens over 4096 cached), one run",
                       "c3": "2 of the 16 sequences, tokens/s over their suffix tokens",
                       "c4": "4 of the 64 sequences, one decode step each",
                       "c5": "one layer of the stack on the 128 suffix tokens, time scaled by the layer count"}[name]}


if __name__ == "__main__":
    main()
