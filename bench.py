#!/usr/bin/env python
"""KVarN decode-step benchmark on one MI355X.

Workload (N=1): 32 layers x batch 32 folded into 1024 sequences, 32 query / 8 kv heads,
head_dim 128, 32768-token context held as a 2-bit KVarN body plus a bf16 residual; bf16 q.
One step = the whole hot path for one new token of every sequence in every layer:
kvarn_append_token (copy into the residual, and the VarN quantization of full residuals into
the body when due) followed by kvarn_decode_attention over all 32 layers' heads.  The residual
is pre-filled so that one flush (16384 tiles quantized) falls inside the timed steps; with the
default 128 steps that is the steady-state mix of one flush per 128 generated tokens.

Prints one JSON line.  value = decode tokens/s = 32 sequences x steps / wall time, with the
fp32 aux format.  The default run then repeats the measurement with the paper's compact aux
format (2.25 bits/element at 2 bits), in a child process of its own, and reports it beside the
main figures as "compact_aux".
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "decode-attn tokens/s + quantize GB/s over 2-bit KVarN cache; % of HBM roofline"
HBM_PEAK_GBS = 8000.0
# Quantizer roofline: algorithmic fp32 ops per element at K = 8 (FWHT 8, initial statistics 6,
# 6 per VarN iteration -- a column and a row variance, two passes each, with the current scale
# factors inside the multiply-adds -- balance + RTN + pack 9) against the VALU issue rate without
# packed math (256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz).
QUANT_OPS_PER_ELEM = 8 + 6 + 6 * 8 + 9
VALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=128,
                    help="timed steps (default 128: one residual flush per 128 steps, as in steady state)")
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="throughput",
                    help="throughput (default), llama, stress, gqa8, tiny, streaming, or accumulation")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-compact", action="store_true",
                    help="skip the second measurement of the throughput workload with the compact aux format")
    ap.add_argument("--cpu-seconds", type=float, default=15.0, help="target wall time of the oracle sample")
    ap.add_argument("--bits", type=int, default=None,
                    help="code width (2 or 4; default: the workload's, 2 for all of them)")
    ap.add_argument("--aux", choices=["f32", "compact"], default="f32",
                    help="aux format of the tiles: fp32 vectors (default) or the compact E4M3/binary16 one")
    ap.add_argument("--stream-tokens", type=int, default=None,
                    help="tokens generated by --workload streaming (default: the workload's 32768)")
    ap.add_argument("--paged", action="store_true",
                    help="move the cache into a randomly permuted pool behind a block table (paged layout)")
    ap.add_argument("--sink", type=int, default=0, help="bf16 sink tokens per sequence (default 0)")
    ap.add_argument("--no-len-hint", action="store_true",
                    help="append without the lock-step length hint (host_len_before = -1): the flush kernel runs "
                         "every step and decides on the device")
    ap.add_argument("--separate-append", action="store_true",
                    help="streaming: kvarn_append_token and kvarn_decode_attention as two calls on every step "
                         "instead of kvarn_append_decode (which appends inside the decode launch)")
    ap.add_argument("--calib-copy-gib", type=float, default=0.0,
                    help="after the run, copy this many GiB device-to-device (a known-size reference for "
                         "hardware byte counters)")
    return ap.parse_args()


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU only; --gpus must be 1",
                          "n_gpus": args.gpus}), flush=True)
        sys.exit(2)
    import numpy as np
    import torch

    from paper_2606_03458_amd import datagen, workloads
    from paper_2606_03458_amd import kvarn as K

    torch.cuda.set_device(0)
    dev = "cuda:0"
    name = args.workload
    if name == "streaming":
        streaming(args)
        return
    if name == "accumulation":
        accumulation(args)
        return
    spec = datagen.WORKLOADS[name]
    seed = datagen.SEEDS[name]
    aux = 1 if args.aux == "compact" else 0
    r = run_steps(args, name, aux, args.paged, args.sink)
    built, length, qs, scale = r["built"], r["length"], r["qs"], r["scale"]
    p = built.params
    n_seq = built.cache.batch
    tb = K.kvarn_tile_bytes(p)
    stream = torch.cuda.current_stream()
    W, S = args.warmup, args.steps
    tokens_per_s, elapsed, dec_avg_s = r["tokens_per_s"], r["elapsed"], r["dec_avg_s"]
    bytes_avg, achieved = r["bytes_avg"], r["achieved"]

    # ---- quantize throughput: one layer's keys (8 kv heads x 32 sequences x 256 tiles) --------
    q_res = None
    try:
        sig = datagen.channel_log_scales(seed * 1000, spec["n_kv"], spec["dist"], device=dev)
        Kx, _ = datagen.kv_tokens(seed * 1000 + 999, 0, spec["batch"], spec["n_kv"], spec["context"], spec["dist"],
                                  dtype=torch.bfloat16, device=dev, sigma_c=sig)
        x = Kx.view(-1, spec["context"], 128)
        n_tiles = x.shape[0] * (spec["context"] // 128)
        body = torch.empty((x.shape[0], spec["context"] // 128, tb), dtype=torch.uint8, device=dev)
        assert tb == K.kvarn_tile_bytes(p)
        K.quantize_into_body(p, K.KVARN_KEYS, x, body)  # warm-up
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        reps = 3
        e0.record(stream)
        for _ in range(reps):
            K.quantize_into_body(p, K.KVARN_KEYS, x, body)
        e1.record(stream)
        torch.cuda.synchronize()
        qt = e0.elapsed_time(e1) / reps / 1e3
        qbytes = n_tiles * (128 * 128 * 2 + tb)
        tops = n_tiles * 128 * 128 * QUANT_OPS_PER_ELEM / qt / 1e12
        q_res = {"value": round(qbytes / qt / 1e9, 2), "unit": "GB/s", "tiles_per_s": round(n_tiles / qt),
                 "tiles": n_tiles, "bytes_per_tile": 128 * 128 * 2 + tb,
                 "frac_hbm": round(qbytes / qt / 1e9 / HBM_PEAK_GBS, 4),
                 "roofline": {"bound": "alu", "achieved": round(tops, 2), "peak": round(VALU_PEAK_TOPS, 1),
                              "unit": "Tops/s", "frac": round(tops / VALU_PEAK_TOPS, 4),
                              "ops_per_element": QUANT_OPS_PER_ELEM, "kernel": "kvarn_quantize_block",
                              "counters": measured_quantizer_counters()}}
        del Kx, x, body
    except Exception as e:  # report, do not hide
        q_res = {"error": repr(e)}

    # ---- CPU baseline: the oracle on a sample of the same streams ------------------------
    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(built, qs[-1], length, scale, args.cpu_seconds)

    # ---- the paper's compact aux format (two E4M3 scales + binary16 offset, 2.25 bits/element at 2 bits)
    # on the same workload, reported beside the fp32-aux figures (default run only) ------------
    compact = None
    if name == "throughput" and aux == 0 and not args.paged and not args.sink and not args.no_compact:
        del r, built, qs
        import gc
        gc.collect()
        torch.cuda.empty_cache()
        # Measured in a process of its own, as the fp32-aux leg is: a second 20-28 GB cache
        # allocated in memory that the first one freed decodes 1-2 % slower than the same cache in
        # a fresh process.  The child is this script with --aux compact; its line is kept whole.
        import subprocess
        cmd = [sys.executable, os.path.abspath(__file__), "--aux", "compact", "--no-cpu-baseline", "--no-compact",
               "--steps", str(S), "--warmup", str(W)]
        if args.bits:
            cmd += ["--bits", str(args.bits)]
        if args.no_len_hint:
            cmd += ["--no-len-hint"]
        try:
            child = subprocess.run(cmd, stdout=subprocess.PIPE, text=True, timeout=900)
            if child.returncode != 0:
                raise RuntimeError(f"the child process ended with status {child.returncode}")
            d = json.loads(child.stdout.strip().splitlines()[-1])
            compact = {"value": d["value"], "unit": "tokens/s", "ms_per_step": d["ms_per_step"],
                       "aux": f"compact ({d['config']['bits'] + 0.25:g} bits/element)",
                       "roofline": {k: d["roofline"][k] for k in ("bound", "achieved", "peak", "unit", "frac",
                                                                  "traffic", "alg_bytes_per_launch", "avg_launch_ms")},
                       "measured_in": "a child process (bench.py --aux compact)"}
        except Exception as e:  # report, do not hide; the main figures stand on their own
            compact = {"error": repr(e)}

    line = {
        "metric": METRIC, "value": round(tokens_per_s, 2), "unit": "tokens/s", "n_gpus": 1, "steps": S,
        "warmup": W, "ms_per_step": round(elapsed / S * 1e3, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "fp32", "data": "synthetic",
        "config": {"workload": f"{name}: {spec['layers']} layers x batch {spec['batch']} = {n_seq} sequences, "
                               f"{spec['n_q']} q / {spec['n_kv']} kv heads, head_dim 128, "
                               f"{spec['context']}-token context, {p.bits}-bit KVarN body + bf16 residual, "
                               f"append + decode per step",
                   "layers": spec["layers"], "batch": spec["batch"], "context": spec["context"], "bits": p.bits,
                   "aux": args.aux, "paged": bool(args.paged), "sink": args.sink,
                   "len_hint": not args.no_len_hint},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": measured_traffic(name, aux, p.bits) if not (args.paged or args.sink) else None,
                     "kernel": "kvarn_decode_attention", "alg_bytes_per_launch": int(bytes_avg),
                     "avg_launch_ms": round(dec_avg_s * 1e3, 4)},
        "cpu_baseline": cpu,
        "quantize": q_res,
    }
    if compact is not None:
        line["compact_aux"] = compact
    print(json.dumps(line), flush=True)

    if args.calib_copy_gib > 0:
        nbytes = int(args.calib_copy_gib * (1 << 30))
        src = torch.empty(nbytes, dtype=torch.uint8, device=dev).fill_(1)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        print(f"[bench] calibration copy: {nbytes} bytes read + {nbytes} bytes written", file=sys.stderr, flush=True)


def run_steps(args, name, aux, paged, sink):
    """Build the workload, pre-fill the residual through the append path and time W + S steps
    of kvarn_append_token + kvarn_decode_attention (inputs of every step drawn before timing)."""
    import numpy as np
    import torch

    from paper_2606_03458_amd import datagen, workloads
    from paper_2606_03458_amd import kvarn as K

    dev = "cuda:0"
    spec = datagen.WORKLOADS[name]
    seed = datagen.SEEDS[name]
    W, S = args.warmup, args.steps
    # residual fill so that one flush lands in the middle of the timed steps
    r0 = (128 - W - max(S // 2, 1)) % 128
    total_tokens = spec["context"] + r0 + W + S
    extra = (total_tokens - spec["context"] + 127) // 128 + 1
    print(f"[bench] building {name} (aux {aux}): {spec}", file=sys.stderr, flush=True)
    t0 = time.time()
    built, _ = workloads.build(name, device=dev, extra_blocks=extra, aux=aux, n_sink=sink, bits=args.bits)
    if paged:
        built.cache = to_paged(K, built.params, built.cache, seed)
    p, cache = built.params, built.cache
    n_seq = cache.batch
    length = built.length
    for t in range(r0):  # pre-fill the residual through the append path
        kt, vt = workloads.step_tokens(built, seed, -1 - t)
        K.kvarn_append_token(p, cache, kt, vt, K.KVARN_BF16, length)
        length += 1
    torch.cuda.synchronize()
    print(f"[bench] built in {time.time() - t0:.1f}s; length {length}, max_blocks {cache.max_blocks}",
          file=sys.stderr, flush=True)

    toks = [workloads.step_tokens(built, seed, s) for s in range(W + S)]
    qs = [workloads.decode_queries(built, seed, s) for s in range(W + S)]
    scale = 1.0 / np.sqrt(128.0)
    max_len = total_tokens + 1
    ws_bytes = K.kvarn_decode_workspace_bytes(p, cache, built.n_q, max_len)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    out = torch.empty_like(qs[0])
    stream = torch.cuda.current_stream()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(S)]
    tb = K.kvarn_tile_bytes(p)

    def decode_bytes(L):
        nb = L // 128
        nr = L % 128
        per_stream = nb * 2 * tb + nr * 2 * 128 * 2
        return n_seq * spec["n_kv"] * per_stream + 2 * n_seq * built.n_q * 128 * 2

    alg_bytes = []
    for s in range(W + S):
        kt, vt = toks[s]
        K.kvarn_append_token(p, cache, kt, vt, K.KVARN_BF16, -1 if args.no_len_hint else length)
        length += 1
        if s == W:
            torch.cuda.synchronize()
            t_start = time.perf_counter()
        if s >= W:
            ev[s - W][0].record(stream)
        K.kvarn_decode_attention(p, cache, built.n_q, qs[s], K.KVARN_BF16, out, K.KVARN_BF16, scale, max_len, ws,
                                 ws_bytes)
        if s >= W:
            ev[s - W][1].record(stream)
            alg_bytes.append(decode_bytes(length))
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t_start
    if not bool(torch.isfinite(out).all()):
        raise RuntimeError("decode output has non-finite values")
    dec_ms = [a.elapsed_time(b) for a, b in ev]
    dec_avg_s = sum(dec_ms) / len(dec_ms) / 1e3
    bytes_avg = sum(alg_bytes) / len(alg_bytes)
    achieved = bytes_avg / dec_avg_s / 1e9
    tokens_per_s = spec["batch"] * S / elapsed
    print(f"[bench] {S} steps in {elapsed * 1e3:.2f} ms; decode avg {dec_avg_s * 1e3:.3f} ms, "
          f"{achieved:.0f} GB/s", file=sys.stderr, flush=True)
    return {"built": built, "length": length, "qs": qs, "scale": scale, "tokens_per_s": tokens_per_s,
            "elapsed": elapsed, "dec_avg_s": dec_avg_s, "bytes_avg": bytes_avg, "achieved": achieved,
            "bits": built.params.bits}


def accumulation(args, layers=4, batch=4, T=2048):
    """Error accumulation through depth and time (Sec. 3.2 and 3.4): a random residual attention
    stack decoded token by token through the library, static (prefill-like) vs dynamic
    (pseudo-decode), KIVI-style RTN vs KVarN.  Prints the last layer's mean relative
    attention-output error per 256-token window and the dynamic error per layer."""
    import torch

    from paper_2606_03458_amd import pseudo_decode as PD

    st = PD.make_stack(layers, batch, T, device="cuda:0")
    ref = PD.reference(st)
    bits = args.bits or 2
    results, win = {}, 256
    for name in PD.QUANTIZERS:
        t0 = time.time()
        err = PD.run(st, ref, name, bits)
        torch.cuda.synchronize()
        print(f"accumulation: {name} done in {time.time() - t0:.1f} s", file=sys.stderr, flush=True)
        results[name] = {m: [round(float(e[layers - 1, i:i + win].mean()), 5) for i in range(0, T, win)]
                         for m, e in err.items()}
        results[name]["dynamic_by_layer"] = [round(float(err["dynamic"][l].mean()), 5) for l in range(layers)]
        results[name]["static_by_layer"] = [round(float(err["static"][l].mean()), 5) for l in range(layers)]
    line = {"metric": "relative error of the attention output, last layer, mean per 256-token window",
            "config": {"workload": f"random residual attention stack: {layers} layers, batch {batch}, {T} tokens, "
                                   f"32 q / 8 kv heads of 128, d_model 1024, {bits}-bit, append + decode per token"},
            "windows": list(range(0, T, win)), "results": results}
    print(json.dumps(line), flush=True)


def to_paged(K, p, cache, seed):
    """The same cache with its body tiles moved to a randomly permuted pool of
    batch * max_blocks blocks behind a block table."""
    import torch
    B, H, MB = cache.batch, cache.n_kv, cache.max_blocks
    paged = K.Cache(p, B, H, MB, device=cache.k_body.device, n_phys=B * MB)
    perm = torch.randperm(B * MB, generator=torch.Generator().manual_seed(seed)).to(cache.k_body.device)
    paged.block_table.copy_(perm.view(B, MB).to(torch.int32))
    for src, dst in ((cache.k_body, paged.k_body), (cache.v_body, paged.v_body)):
        flat = src.permute(0, 2, 1, 3).reshape(B * MB, H, -1)  # [(b, blk)][kv head][tile]
        dst.index_copy_(0, perm, flat)
        del flat
    for f in ("k_resid", "v_resid", "k_sink", "v_sink", "seq_len"):
        if getattr(cache, f) is not None:
            getattr(paged, f).copy_(getattr(cache, f))
    del cache
    return paged


def streaming(args):
    """Streaming pseudo-decode from an empty cache: 64 sequences x 8 kv heads (32 q heads)
    each generate one token per step; every step appends the token (a residual reaching 128
    tokens is quantized into a body tile) and decodes over the whole cache, in one
    kvarn_append_decode call on the steps that do not flush.  Prints one JSON line: tokens/s
    from GPU time, per-step time against context, the quantize share."""
    import ctypes

    import numpy as np
    import torch

    from paper_2606_03458_amd import datagen
    from paper_2606_03458_amd import kvarn as K

    dev = "cuda:0"
    spec = datagen.WORKLOADS["streaming"]
    seed = datagen.SEEDS["streaming"]
    bits = args.bits or spec["bits"]
    B, n_kv, n_q = spec["batch"], spec["n_kv"], spec["n_q"]
    T = args.stream_tokens or spec["context"]
    p = K.kvarn_params_init(bits)
    p.aux_format = 1 if args.aux == "compact" else 0
    cache = K.Cache(p, B, n_kv, (T + 127) // 128 + 1, device=dev)
    sig = datagen.channel_log_scales(seed * 1000, n_kv, spec["dist"], device=dev)
    Kx, Vx = datagen.kv_tokens(seed * 1000, 0, B, n_kv, T, spec["dist"], dtype=torch.bfloat16, device=dev,
                               sigma_c=sig)
    Kt = Kx.permute(2, 0, 1, 3).contiguous()  # [T, B, n_kv, 128]: one contiguous token per step
    del Kx
    Vt = Vx.permute(2, 0, 1, 3).contiguous()
    del Vx
    qpool = [datagen.queries(seed, s, B, n_q, dtype=torch.bfloat16, device=dev) for s in range(16)]
    out = torch.empty_like(qpool[0])
    ws_bytes = max(K.kvarn_decode_workspace_bytes(p, cache, n_q, L) for L in range(1, T + 2, 64))
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device=dev)
    scale = 1.0 / np.sqrt(128.0)
    tb = K.kvarn_tile_bytes(p)

    L = K.lib()
    d = cache.desc()
    pp, dd = ctypes.byref(p), ctypes.byref(d)
    stream = torch.cuda.current_stream()
    sp = stream.cuda_stream
    kptr = [Kt[t].data_ptr() for t in range(T)]
    vptr = [Vt[t].data_ptr() for t in range(T)]
    qptr = [q.data_ptr() for q in qpool]
    optr, wptr = out.data_ptr(), ws.data_ptr()
    n_blk = (T + 127) // 128
    ev_blk = [torch.cuda.Event(enable_timing=True) for _ in range(n_blk + 1)]
    ev_fl = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(T // 128)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for t in range(T):
        if t % 128 == 0:
            ev_blk[t // 128].record(stream)
        flush = t % 128 == 127
        if flush:
            ev_fl[t // 128][0].record(stream)
        if flush or args.separate_append:  # the flush step keeps its own timing
            st = L.kvarn_append_token(pp, dd, kptr[t], vptr[t], K.KVARN_BF16, t, sp)
            if flush:
                ev_fl[t // 128][1].record(stream)
            st |= L.kvarn_decode_attention(pp, dd, n_q, qptr[t % 16], K.KVARN_BF16, optr, K.KVARN_BF16, scale,
                                           t + 1, wptr, ws_bytes, sp)
        else:
            st = L.kvarn_append_decode(pp, dd, kptr[t], vptr[t], K.KVARN_BF16, t, n_q, qptr[t % 16], K.KVARN_BF16,
                                       optr, K.KVARN_BF16, scale, wptr, ws_bytes, sp)
        if st:
            raise RuntimeError(f"step {t}: status {st}")
    ev_blk[n_blk].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    if int(cache.err_word.item()) != 0 or not bool(torch.isfinite(out).all()):
        raise RuntimeError("streaming run left an error flag or a non-finite output")
    blk_ms = [ev_blk[i].elapsed_time(ev_blk[i + 1]) for i in range(n_blk)]
    gpu_s = sum(blk_ms) / 1e3
    flush_ms = [a.elapsed_time(b) for a, b in ev_fl]
    streams = B * n_kv

    def step_bytes(length):  # decode after the append of token length - 1
        nb, nr = length // 128, length % 128
        return streams * (nb * 2 * tb + nr * 2 * 256) + 2 * B * n_q * 128 * 2 + streams * 2 * 256 * 2

    alg = sum(step_bytes(t + 1) for t in range(T)) + (T // 128) * streams * 2 * (128 * 128 * 2 + tb)
    at = {f"{k // 1024}k": round(blk_ms[k // 128 - 1] / 128, 4) for k in (1024, 4096, 8192, 16384, 32768)
          if k // 128 - 1 < n_blk}
    line = {"metric": "streaming pseudo-decode tokens/s (append + flush + decode per step)",
            "value": round(B * T / gpu_s, 1), "unit": "tokens/s", "n_gpus": 1, "steps": T,
            "higher_is_better": True, "dtype": "fp32", "data": "synthetic",
            "config": {"workload": f"streaming: batch {B}, {n_q} q / {n_kv} kv heads, head_dim 128, {T} tokens "
                                   f"from an empty cache, {bits}-bit, flush every 128", "bits": bits,
                       "aux": args.aux, "step": "two calls" if args.separate_append else "kvarn_append_decode"},
            "gpu_s": round(gpu_s, 4), "wall_s": round(wall, 3),
            "ms_per_step_at_context": at,
            "alg_GBps": round(alg / gpu_s / 1e9, 1),
            "quantize_share": round(sum(flush_ms) / 1e3 / gpu_s, 5),
            "flush_ms_avg": round(sum(flush_ms) / max(len(flush_ms), 1), 4)}
    print(json.dumps(line), flush=True)


PROFILES = os.path.join(ROOT, "profiles")
DECODE_SOURCES = [os.path.join(ROOT, "paper_2606_03458_amd", "csrc", f) for f in ("decode.hip", "common.hpp", "plan.hpp")]
QUANT_SOURCES = [os.path.join(ROOT, "paper_2606_03458_amd", "csrc", f) for f in ("quantize.hip", "common.hpp")]


def source_hash(files) -> str:
    import hashlib
    h = hashlib.sha256()
    for f in files:
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def decode_source_hash() -> str:
    return source_hash(DECODE_SOURCES)


def _summary_fields(path):
    """`key: value` lines of a committed profile summary."""
    fields = {}
    try:
        with open(path) as fh:
            for line in fh:
                line = line.strip().strip("`")
                if ":" in line and " " not in line.split(":", 1)[0]:
                    k, v = line.split(":", 1)
                    fields.setdefault(k, v.strip())
    except OSError:
        pass
    return fields


def measured_traffic(workload: str, aux: int = 0, bits: int = 2):
    """HBM bytes per decode launch (FETCH_SIZE + WRITE_SIZE, calibrated) from the committed
    rocprofv3 counter summaries (profiles/*_hbm_counters.md); None unless one covers this
    workload, aux format and code width and was taken on the current decode sources."""
    import glob
    want = decode_source_hash()
    for path in sorted(glob.glob(os.path.join(PROFILES, "*decode*_hbm_counters.md"))):
        f = _summary_fields(path)
        if (f.get("workload"), f.get("aux", "0"), f.get("bits", "2"), f.get("source_sha256")) == \
                (workload, str(aux), str(bits), want):
            try:
                return int(f["hbm_bytes_per_launch"])
            except (KeyError, ValueError):
                return None
    return None


def measured_quantizer_counters():
    """VALU instructions per element and VALU-busy fraction of k_quantize_tiles from the
    committed counter summary, while the quantizer sources hash to the profiled ones."""
    f = _summary_fields(os.path.join(PROFILES, "k_quantize_tiles_valu_counters.md"))
    if f.get("source_sha256") != source_hash(QUANT_SOURCES):
        return None
    try:
        return {"valu_insts_per_element": float(f["valu_insts_per_element"]),
                "valu_busy": float(f["valu_busy"]), "source": "profiles/k_quantize_tiles_valu_counters.md"}
    except (KeyError, ValueError):
        return None


def cpu_model() -> str:
    """The host's CPU model name, with family / model / stepping (a virtualized host may report
    only a generic name), from /proc/cpuinfo."""
    fields = {}
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if not line.strip():
                    break  # the first processor's block is enough
                k, _, v = line.partition(":")
                fields[k.strip()] = v.strip()
    except OSError:
        return "unknown"
    name = fields.get("model name", "unknown")
    ids = [f"{k} {fields[k]}" for k in ("cpu family", "model", "stepping") if k in fields]
    return f"{name} ({', '.join(ids)})" if ids else name


def cpu_baseline(built, q, length, scale, target_s):
    """Time the oracle's decode on a sample of (sequence, kv head) streams of the same cache,
    scaled to the metric's unit (tokens/s of the whole 1024-sequence step)."""
    import numpy as np

    import oracle

    cache = built.cache
    n_kv = cache.n_kv
    g = built.n_q // n_kv
    total_streams = cache.batch * n_kv
    rng = np.random.default_rng(0)

    def sample(n):
        idx = rng.choice(total_streams, size=n, replace=False)
        hc = oracle.HostCache(n, 1, cache.max_blocks, bits=cache.bits, aux=cache.aux, rotate=cache.rotate)
        qh = np.zeros((n, g, 128), dtype=np.uint16)
        for i, s in enumerate(idx):
            b, kh = divmod(int(s), n_kv)
            hc.k_body[i, 0] = cache.k_body[b, kh].cpu().numpy()
            hc.v_body[i, 0] = cache.v_body[b, kh].cpu().numpy()
            hc.k_resid[i, 0] = cache.k_resid[b, kh].view(torch_int16()).cpu().numpy().view(np.uint16)
            hc.v_resid[i, 0] = cache.v_resid[b, kh].view(torch_int16()).cpu().numpy().view(np.uint16)
            hc.seq_len[i] = int(cache.seq_len[b])
            qh[i] = q[b, kh * g:(kh + 1) * g].view(torch_int16()).cpu().numpy().view(np.uint16)
        return hc, qh

    hc, qh = sample(1)
    t0 = time.perf_counter()
    oracle.decode(hc, qh, scale)
    one = time.perf_counter() - t0
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    n = int(max(1, min(total_streams, target_s / one * threads)))
    n = max(threads, (n // threads) * threads) if n >= threads else n
    hc, qh = sample(n)
    t0 = time.perf_counter()
    oracle.decode(hc, qh, scale)
    t = time.perf_counter() - t0
    step_s = t * total_streams / n
    # the same on one thread, over a smaller sample (about a fifth of the time budget)
    n1 = int(max(1, min(total_streams, target_s / 5 / one)))
    hc1, qh1 = sample(n1)
    oracle.set_threads(1)
    try:
        t0 = time.perf_counter()
        oracle.decode(hc1, qh1, scale)
        t1 = time.perf_counter() - t0
    finally:
        oracle.set_threads(threads)
    return {"value": round(built.spec["batch"] / step_s, 4), "unit": "tokens/s", "cores": min(threads, n),
            "kind": "oracle", "cpu_model": cpu_model(), "host_threads": os.cpu_count(),
            "sample": f"{n} of {total_streams} (sequence, kv head) streams at length {int(hc.seq_len[0])}, "
                      f"decode only, {t:.1f} s wall, scaled linearly to the full step",
            "single_thread": {"value": round(built.spec["batch"] / (t1 * total_streams / n1), 4), "unit": "tokens/s",
                              "sample": f"{n1} streams, {t1:.1f} s wall on 1 thread, scaled linearly"}}


def torch_int16():
    import torch
    return torch.int16


if __name__ == "__main__":
    main()
