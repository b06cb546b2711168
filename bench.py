#!/usr/bin/env python3
"""Benchmark of the QK4PV8 attention hot path on one MI355X.

One step = the whole path over one batch of synthetic input:
  * quantization / cache-write pass of the 128K-token Qwen3-14B-shaped causal
    prefill (statistics, NVFP4 Q/K, FP8 V, Delta_S),
  * the causal prefill over it (the headline: attention TFLOP/s),
  * split-KV paged decode of the Llama-3.1-8B-shaped batch (32 sequences,
    contexts U[16384, 131072]) over a pre-quantized, shuffled 64-token-page
    cache (decode KV GB/s).
Inputs are resident in HBM before the timed region; kernel times come from
HIP events on the stream the kernels run on.  Prints one JSON line.
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

PEAK_FP4 = 10.1e15        # MI355X dense MXFP4 / FP4 FLOP/s (published)
PEAK_FP8 = 5.0e15         # dense FP8
PEAK_BF16 = 2.5e15        # dense BF16 / FP16
PEAK_HBM = 8.0e12         # bytes/s

# HBM bytes per launch measured with rocprofv3 FETCH_SIZE / WRITE_SIZE passes,
# scaled by what the same counters read for a plain device copy.  A figure is
# reported only while the kernel's sources hash to the value recorded with it.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "pmc_traffic.txt")
KERNEL_SOURCES = {
    "prefill_kernel": ["csrc/prefill.hip", "csrc/prefill_body.h", "csrc/prefill_split.h", "csrc/mpfa_device.h", "csrc/mpfa_internal.h",
                       "csrc/api.cpp"],
    "decode_kernel": ["csrc/decode.hip", "csrc/decode_body.h", "csrc/mpfa_device.h", "csrc/mpfa_internal.h",
                      "csrc/api.cpp"],
}


def source_hash(kernel: str) -> str:
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(ROOT, "paper_2609_33135_amd", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(kernel: str):
    """HBM bytes per launch of `kernel` from the committed counter summary, or None
    when there is none or the kernel's sources changed since it was taken."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    kv = {}
    with open(TRAFFIC_FILE) as fh:
        for line in fh:
            line = line.split("#", 1)[0].strip()
            if "=" in line:
                k, v = (x.strip() for x in line.split("=", 1))
                kv[k] = v
    try:
        if kv[f"{kernel}.source_sha256"] != source_hash(kernel):
            return None
        kib = 1024.0
        return (float(kv[f"{kernel}.fetch_kib"]) * float(kv["fetch_factor"])
                + float(kv[f"{kernel}.write_kib"]) * float(kv["write_factor"])) * kib
    except KeyError:
        return None


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--prefill-seq", type=int, default=131072)
    ap.add_argument("--decode-batch", type=int, default=32)
    ap.add_argument("--no-prefill", action="store_true")
    ap.add_argument("--no-decode", action="store_true")
    ap.add_argument("--no-direct", action="store_true", help="skip the unsmoothed prefill variant")
    ap.add_argument("--no-mxfp4", action="store_true", help="skip the MXFP4 variant runs")
    ap.add_argument("--no-mixed", action="store_true",
                    help="skip the mixed serving step (separate launches vs one fused launch)")
    ap.add_argument("--no-decode128k", action="store_true",
                    help="skip the decode batch whose contexts are all 131072 tokens")
    ap.add_argument("--no-peaks", action="store_true",
                    help="skip the measurement of achievable GEMM and copy rates on this GPU")
    ap.add_argument("--no-sweep", action="store_true",
                    help="skip the Llama-shaped prefill length sweep (16K, 32K, 64K tokens)")
    ap.add_argument("--no-precision", action="store_true",
                    help="skip the BF16 / NVFP4 PV precision-assignment runs")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-accuracy", action="store_true",
                    help="skip the error report against FP64 unquantized attention")
    ap.add_argument("--cpu-rows", type=int, default=16384, help="oracle sample: query rows of head 0")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB device copy (reference for memory counters)")
    ap.add_argument("--ablation", action="store_true",
                    help="softmax ablation chain of the prefill (characterization library): exp2 off, "
                         "then row max / row sum / rescale off")
    return ap.parse_args()


class Timer:
    """HIP events on the current stream around a region."""

    def __init__(self, torch):
        self.t = torch
        self.s = torch.cuda.Event(enable_timing=True)
        self.e = torch.cuda.Event(enable_timing=True)

    def __enter__(self):
        self.s.record()
        return self

    def __exit__(self, *exc):
        self.e.record()

    def ms(self):
        self.e.synchronize()
        return self.s.elapsed_time(self.e)


def measured_peaks(torch):
    """Achievable rates of this GPU, as a second denominator beside the
    specification: large square GEMMs through torch (hipBLASLt) in FP16, BF16
    and, where torch offers it, FP8 E4M3 with unit scales; and a 1 GiB device
    copy (bytes read + written per second).  Context for the rooflines, not a
    product path."""
    out = {}
    n = 8192

    def timed(fn, reps=10):
        for _ in range(2):
            fn()
        torch.cuda.synchronize()
        with Timer(torch) as t:
            for _ in range(reps):
                fn()
        return t.ms() / reps

    for name, dt in (("fp16_gemm_tflops", torch.float16), ("bf16_gemm_tflops", torch.bfloat16)):
        a = torch.randn(n, n, device="cuda").to(dt)
        b = torch.randn(n, n, device="cuda").to(dt)
        ms = timed(lambda: torch.matmul(a, b))
        out[name] = 2.0 * n ** 3 / (ms * 1e-3) / 1e12
        del a, b
    try:
        a = torch.randn(n, n, device="cuda").to(torch.float8_e4m3fn)
        b = torch.randn(n, n, device="cuda").to(torch.float8_e4m3fn).t()
        one = torch.ones((), device="cuda")
        ms = timed(lambda: torch._scaled_mm(a, b, scale_a=one, scale_b=one, out_dtype=torch.bfloat16))
        out["fp8_gemm_tflops"] = 2.0 * n ** 3 / (ms * 1e-3) / 1e12
        del a, b
    except Exception as e:   # FP8 GEMM not available in this torch build
        out["fp8_gemm_tflops"] = None
        out["fp8_gemm_note"] = f"unavailable: {type(e).__name__}"
    src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    ms = timed(lambda: dst.copy_(src), reps=5)
    out["copy_GBps"] = 2.0 * (1 << 30) / (ms * 1e-3) / 1e9
    out["note"] = ("library rates on this stack (torch.matmul / _scaled_mm through hipBLASLt, "
                   "8192^3; torch copy_ of 1 GiB, read + write bytes), not hardware peaks")
    del src, dst
    torch.cuda.empty_cache()
    return out


def probe_peaks(torch, mp):
    """Achievable rates measured by the probe kernels (libmpfa_probe.so): each MFMA
    form the attention kernels use, issued back to back by 8 waves per SIMD
    (2048 workgroups, 8 independent accumulators per wave), and the HBM read
    rate of a 4 GiB buffer read once through registers or directly into LDS,
    each workgroup streaming a contiguous share (best of four grid sizes).
    Best of 3 launches each, HIP events."""
    out = {}
    blocks, iters = 2048, 10000
    sink = torch.empty(blocks * 256, dtype=torch.float32, device="cuda")
    for name, kind in (("mfma_f16_tflops", mp.PROBE_MFMA_F16), ("mfma_fp8_tflops", mp.PROBE_MFMA_FP8),
                       ("mfma_fp4_tflops", mp.PROBE_MFMA_FP4)):
        mp.probe_mfma(kind, 10, blocks, sink)
        torch.cuda.synchronize()
        best = None
        for _ in range(3):
            with Timer(torch) as t:
                fl = mp.probe_mfma(kind, iters, blocks, sink)
            ms = t.ms()
            best = ms if best is None else min(best, ms)
        out[name] = fl / (best * 1e-3) / 1e12
    del sink
    nbytes = 1 << 32
    buf = torch.empty(nbytes // 4, dtype=torch.int32, device="cuda")
    buf.fill_(0x5A5A5A5A)
    for name, mode in (("read_vgpr_GBps", mp.PROBE_READ_VGPR), ("read_lds_GBps", mp.PROBE_READ_LDS)):
        best, best_blocks = None, None
        for nb in (1024, 2048, 4096, 8192):
            sink = torch.empty(nb * 256, dtype=torch.int32, device="cuda")
            mp.probe_read(mode, buf, nb, sink)
            torch.cuda.synchronize()
            for _ in range(3):
                with Timer(torch) as t:
                    mp.probe_read(mode, buf, nb, sink)
                ms = t.ms()
                if best is None or ms < best:
                    best, best_blocks = ms, nb
            del sink
        out[name] = nbytes / (best * 1e-3) / 1e9
        out[name.replace("GBps", "blocks")] = best_blocks
    del buf
    torch.cuda.empty_cache()
    out["note"] = ("probe kernels of libmpfa_probe (mpfa_probe_mfma, mpfa_probe_read): dense MFMA issue "
                   "rate per form and single-pass HBM read rate")
    return out


def setup_prefill(torch, np, mp, W, seq, smooth, mx=False, pv=0, wl=None):
    wl = wl if wl is not None else W.qwen_prefill(seq)
    dev = "cuda"
    q, k, v = W.gen_qkv(wl.seed, [seq], wl.h_q, wl.h_kv, wl.outliers, dev)
    pt, n_pages = W.make_pages(wl.seed, [seq])
    slots = W.slots_for(pt, 0, range(seq))
    d = lambda a: torch.from_numpy(a).to(dev)
    st = dict(wl=wl, q=q, k=k, v=v, pt=pt, pt_d=d(pt), n_pages=n_pages,
              cu=d(np.array([0, seq], np.int32)), slots=d(slots),
              q_start=d(np.zeros(1, np.int32)), kv_len=d(np.array([seq], np.int32)),
              cache=mp.PagedCache(n_pages, wl.h_q, wl.h_kv, dev, smooth=smooth, pv=pv),
              stats=mp.SeqStats(1, wl.h_q, wl.h_kv, dev), qq=mp.QuantQ(seq, 1, wl.h_q, dev),
              out=torch.empty((seq, wl.h_q, 128), dtype=torch.bfloat16, device=dev),
              flags=(mp.SMOOTH if smooth else 0) | (mp.MXFP4 if mx else 0) | pv)
    return st


def run_quant(mp, st):
    mp.quantize_qk(st["q"], st["k"], st["v"], st["cu"], st["slots"], st["cache"], st["stats"],
                   st["qq"], st["flags"] | mp.COMPUTE_STATS, st["q"].shape[0])


def run_prefill(mp, st):
    mp.prefill(st["qq"], st["cache"], st["stats"], st["cu"], st["q_start"], st["kv_len"],
               st["pt_d"], st["out"], st["q"].shape[0], st["flags"])


def setup_decode(torch, np, mp, W, batch, mx=False, smooth=True, ctx_range=None):
    wl = W.llama_decode(batch) if ctx_range is None else W.llama_decode(batch, *ctx_range)
    dev = "cuda"
    fmt = (mp.MXFP4 if mx else 0) | (mp.SMOOTH if smooth else 0)
    lens = wl.kv_len
    pt, n_pages = W.make_pages(wl.seed, lens)
    cache = mp.PagedCache(n_pages, wl.h_q, wl.h_kv, dev, smooth=smooth)
    stats = mp.SeqStats(batch, wl.h_q, wl.h_kv, dev)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    # context cache write per sequence (statistics over the context, then frozen)
    for b, n in enumerate(lens):
        ctx = n - 1
        q, k, v = W.gen_qkv(wl.seed, [ctx], wl.h_q, wl.h_kv, wl.outliers, dev, seq_ids=[b])
        sb = mp.SeqStats(1, wl.h_q, wl.h_kv, dev)
        qq = mp.QuantQ(ctx, 1, wl.h_q, dev)
        slots = W.slots_for(pt, b, range(ctx))
        mp.quantize_qk(q, k, v, d(np.array([0, ctx], np.int32)), d(slots), cache, sb, qq,
                       mp.COMPUTE_STATS | fmt, ctx)
        stats.q_mean[b].copy_(sb.q_mean[0])
        stats.k_mean[b].copy_(sb.k_mean[0])
        stats.k_tscale[b].copy_(sb.k_tscale[0])
        del q, k, v, qq
    torch.cuda.synchronize()
    # the new token of every sequence: appended (frozen statistics), then queried
    qn, kn, vn = W.gen_qkv(wl.seed, [1] * batch, wl.h_q, wl.h_kv, wl.outliers, dev,
                           tok_offsets=[n - 1 for n in lens])
    slots1 = np.array([W.slots_for(pt, b, [lens[b] - 1])[0] for b in range(batch)], np.int64)
    qq = mp.QuantQ(batch, batch, wl.h_q, dev)
    mp.quantize_qk(qn, kn, vn, d(np.arange(batch + 1, dtype=np.int32)), d(slots1), cache,
                   stats, qq, fmt, 1)
    part = mp.decode_choose_partition(lens, wl.h_kv, torch.cuda.get_device_properties(0).multi_processor_count)
    maxp = max(math.ceil(n / part) for n in lens)
    ws = torch.empty(mp.decode_workspace_size(batch, wl.h_q, maxp) // 4, dtype=torch.float32,
                     device=dev)
    out = torch.empty((batch, wl.h_q, 128), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    return dict(wl=wl, lens=lens, pt=pt, pt_d=d(pt), cache=cache, stats=stats, qq=qq, ws=ws,
                out=out, kv_len=d(np.asarray(lens, np.int32)), part=part, maxp=maxp,
                flags=fmt, mx=mx, smooth=smooth)


def run_decode(mp, st):
    mp.decode_paged(st["qq"], st["cache"], st["stats"], st["kv_len"], st["pt_d"], st["out"],
                    st["part"], st["maxp"], st["ws"], st["flags"])


def decode_graph_replay(torch, mp, st, steps, warmup):
    """The decode step (partition kernel + merge) captured once in a HIP graph
    and replayed, as a serving loop runs it (the split-KV workspace is
    preallocated, Sec. 5.3 / Sec. 6).  Reports whether the replayed output
    equals the eager launch's bytes."""
    run_decode(mp, st)
    torch.cuda.synchronize()
    want = st["out"].clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run_decode(mp, st)
    torch.cuda.synchronize()
    for _ in range(max(warmup, 1)):
        g.replay()
    torch.cuda.synchronize()
    identical = torch.equal(st["out"].view(torch.int16), want.view(torch.int16))
    if not identical:
        log("decode graph replay differs from the eager launch")
    ts = []
    for _ in range(steps):
        with Timer(torch) as t:
            g.replay()
        ts.append(t)
    torch.cuda.synchronize()
    ms = sum(t.ms() for t in ts) / steps
    return {"ms": ms, "ms_min": min(t.ms() for t in ts), "GB/s": decode_bytes(st) / (ms * 1e-3) / 1e9,
            "identical_to_eager": identical}


def decode_bytes(st):
    """Algorithmic bytes of one decode launch: K codes + scales + V codes + Delta_S of
    every key (none without smoothing), the quantized queries, the outputs, the
    page-table entries."""
    wl = st["wl"]
    keys = sum(st["lens"])
    scale_bytes = 4 if st.get("mx") else 8       # MXFP4 reads scale bytes 0..3 only
    per_key = wl.h_kv * (64 + scale_bytes + 128) + (wl.h_q * 2 if st.get("smooth", True) else 0)
    pages = sum(math.ceil(n / 64) for n in st["lens"])
    return keys * per_key + wl.batch * wl.h_q * (72 + 4) + wl.batch * wl.h_q * 256 + pages * 4 \
        + wl.batch * 4


def fp64_reference(np, st, n_heads, n_rows):
    """Textbook causal softmax attention in FP64 over the unquantized BF16 inputs
    (Eq. 2) for a sample: `n_heads` query heads spread over the KV heads and
    `n_rows` query rows spread over the sequence (first and last included)."""
    import torch
    q, k, v = st["q"], st["k"], st["v"]
    seq, h_q, h_kv = q.shape[0], q.shape[1], k.shape[1]
    grp = h_q // h_kv
    heads = sorted({(i * h_q) // n_heads for i in range(n_heads)})
    rows = np.unique(np.linspace(0, seq - 1, n_rows).astype(np.int64))
    idx = torch.from_numpy(rows).to(q.device)
    ref = {}
    for h in heads:
        kk = k[:, h // grp].float().cpu().numpy().astype(np.float64)
        vv = v[:, h // grp].float().cpu().numpy().astype(np.float64)
        qq = q[idx, h].float().cpu().numpy().astype(np.float64)
        s = (qq @ kk.T) / math.sqrt(qq.shape[1])
        s[np.arange(seq)[None, :] > rows[:, None]] = -np.inf
        pr = np.exp(s - s.max(axis=1, keepdims=True))
        ref[h] = (pr @ vv) / pr.sum(axis=1, keepdims=True)
    return {"heads": heads, "rows": rows, "idx": idx, "o": ref}


def error_vs_fp64(np, out, ref):
    """Relative L2 and max-abs error of a BF16 output [T, H, 128] on the sampled
    rows of `ref`."""
    rows = ref["idx"].to(out.device)
    num = den = 0.0
    mx = 0.0
    for h in ref["heads"]:
        o = out[rows, h].float().cpu().numpy().astype(np.float64)
        d = o - ref["o"][h]
        num += float((d * d).sum())
        den += float((ref["o"][h] ** 2).sum())
        mx = max(mx, float(np.abs(d).max()))
    return {"rel_l2": math.sqrt(num / den), "max_abs": mx}


def setup_mixed(torch, np, mp, W):
    """The mixed serving step (Qwen shapes): a 32768-token chunk at position
    65536 over its cached prefix, and 64 decode sequences with contexts
    U[8192, 131072] whose caches are written first; then the step's own
    quantization (chunk and new tokens).  Returns the launch arguments."""
    pre, dec = W.mixed_step()
    dev = "cuda"
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    h_q, h_kv = pre.h_q, pre.h_kv
    prefix, chunk = pre.q_start[0], pre.seqlens[0]
    total = prefix + chunk
    pt_pre, np_pre = W.make_pages(pre.seed, [total])
    pt_dec, np_dec = W.make_pages(dec.seed, dec.kv_len)
    pt_dec = pt_dec + np_pre
    cache = mp.PagedCache(np_pre + np_dec, h_q, h_kv, dev)
    st_pre = mp.SeqStats(1, h_q, h_kv, dev)
    qp, kp, vp = W.gen_qkv(pre.seed, [prefix], h_q, h_kv, True, dev)
    mp.quantize_qk(qp, kp, vp, d(np.array([0, prefix], np.int32)), d(W.slots_for(pt_pre, 0, range(prefix))),
                   cache, st_pre, mp.QuantQ(prefix, 1, h_q, dev), mp.SMOOTH | mp.COMPUTE_STATS, prefix)
    del qp, kp, vp
    lens = np.asarray(dec.kv_len)
    ctx = [int(n) - 1 for n in lens]
    st_dec = mp.SeqStats(dec.batch, h_q, h_kv, dev)
    for b0 in range(0, dec.batch, 8):   # contexts in batches of 8 sequences
        ids = list(range(b0, min(b0 + 8, dec.batch)))
        q, k, v = W.gen_qkv(dec.seed, [ctx[b] for b in ids], h_q, h_kv, True, dev, seq_ids=ids)
        cu = np.concatenate([[0], np.cumsum([ctx[b] for b in ids])]).astype(np.int32)
        slots = np.concatenate([W.slots_for(pt_dec, b, range(ctx[b])) for b in ids])
        sb = mp.SeqStats(len(ids), h_q, h_kv, dev)
        mp.quantize_qk(q, k, v, d(cu), d(slots), cache, sb, mp.QuantQ(int(cu[-1]), len(ids), h_q, dev),
                       mp.SMOOTH | mp.COMPUTE_STATS, max(ctx[b] for b in ids))
        for i, b in enumerate(ids):
            st_dec.q_mean[b].copy_(sb.q_mean[i])
            st_dec.k_mean[b].copy_(sb.k_mean[i])
            st_dec.k_tscale[b].copy_(sb.k_tscale[i])
        del q, k, v
    qc, kc, vc = W.gen_qkv(pre.seed, [chunk], h_q, h_kv, True, dev, tok_offsets=[prefix])
    qq_pre = mp.QuantQ(chunk, 1, h_q, dev)
    # the step's own quantization calls (chunk with the frozen prefix statistics,
    # then the decode tokens), kept for the timing that includes them
    quant_chunk = (qc, kc, vc, d(np.array([0, chunk], np.int32)), d(W.slots_for(pt_pre, 0, range(prefix, total))),
                   cache, st_pre, qq_pre, mp.SMOOTH, chunk)
    mp.quantize_qk(*quant_chunk)
    qn, kn, vn = W.gen_qkv(dec.seed, [1] * dec.batch, h_q, h_kv, True, dev, tok_offsets=ctx)
    qq_dec = mp.QuantQ(dec.batch, dec.batch, h_q, dev)
    slots1 = np.array([W.slots_for(pt_dec, b, [ctx[b]])[0] for b in range(dec.batch)], np.int64)
    quant_new = (qn, kn, vn, d(np.arange(dec.batch + 1, dtype=np.int32)), d(slots1), cache, st_dec, qq_dec,
                 mp.SMOOTH, 1)
    mp.quantize_qk(*quant_new)
    part = mp.decode_choose_partition(lens, h_kv, torch.cuda.get_device_properties(0).multi_processor_count)
    maxp = max(math.ceil(n / part) for n in lens)
    pre_args = dict(qq=qq_pre, cache=cache, stats=st_pre, cu_seqlens_q=d(np.array([0, chunk], np.int32)),
                    q_start=d(np.array([prefix], np.int32)), kv_len=d(np.array([total], np.int32)),
                    page_table=d(pt_pre), out=torch.empty((chunk, h_q, 128), dtype=torch.bfloat16, device=dev),
                    max_seqlen_q=chunk)
    dec_args = dict(qq=qq_dec, cache=cache, stats=st_dec, kv_len=d(lens.astype(np.int32)), page_table=d(pt_dec),
                    out=torch.empty((dec.batch, h_q, 128), dtype=torch.bfloat16, device=dev),
                    partition_tokens=part, max_partitions=maxp)
    ws = torch.empty(mp.decode_workspace_size(dec.batch, h_q, maxp) // 4, dtype=torch.float32, device=dev)
    wsm = torch.zeros(mp.mixed_workspace_size(dec.batch, h_q, h_kv, maxp) // 4, dtype=torch.float32, device=dev)
    pairs = sum((prefix + i + 1) for i in range(chunk)) * h_q
    keys = int(lens.sum())
    return dict(pre=pre_args, dec=dec_args, ws=ws, wsm=wsm, pairs=pairs, keys=keys, part=part,
                quant=(quant_chunk, quant_new))


def run_mixed_separate(mp, mx):
    a, b = mx["pre"], mx["dec"]
    mp.prefill(a["qq"], a["cache"], a["stats"], a["cu_seqlens_q"], a["q_start"], a["kv_len"], a["page_table"],
               a["out"], a["max_seqlen_q"], mp.SMOOTH)
    mp.decode_paged(b["qq"], b["cache"], b["stats"], b["kv_len"], b["page_table"], b["out"],
                    b["partition_tokens"], b["max_partitions"], mx["ws"], mp.SMOOTH)


def run_mixed_fused(mp, mx):
    mp.mixed_step(mx["pre"], mx["dec"], mx["wsm"], mp.SMOOTH)


def run_mixed_with_quant(mp, mx):
    """The whole step as a serving engine issues it: quantize the chunk and the
    decode tokens into the cache (rewriting the same slots with the same
    values), then the one-launch attention step."""
    for args in mx["quant"]:
        mp.quantize_qk(*args)
    mp.mixed_step(mx["pre"], mx["dec"], mx["wsm"], mp.SMOOTH)


def quant_bytes(wl, seq):
    """Algorithmic HBM bytes of one quantization / cache-write pass: the
    statistics read Q and K, the quantizer reads Q, K, V and writes the NVFP4 /
    MXFP4 rows (64 code + 8 scale bytes), the FP8 V bytes and Delta_S."""
    row = 128 * 2
    reads = seq * (2 * (wl.h_q + wl.h_kv) * row + wl.h_kv * row)
    writes = seq * (wl.h_q * 72 + wl.h_kv * 72 + wl.h_kv * 128 + wl.h_q * 2)
    return reads + writes


def cpu_baseline(np, W, st, rows):
    """Time the CPU oracle (as it stands) on a bounded sample of the same prefill
    workload: query head 0, `rows` query rows spread over the sequence."""
    from oracle import oracle as orc
    orc.build()
    wl = st["wl"]
    seq = st["q"].shape[0]
    log(f"cpu baseline: oracle quantization of the {seq}-token workload ...")
    ref = orc.quantize_qk(W.bits(st["q"]), W.bits(st["k"]), W.bits(st["v"]),
                          np.array([0, seq], np.int32), W.slots_for(st["pt"], 0, range(seq)),
                          st["n_pages"], orc.SMOOTH | orc.COMPUTE_STATS)
    pos = np.unique(np.linspace(0, seq - 1, rows).astype(np.int64))
    items = np.array([(0, int(i), 0) for i in pos], np.int32)
    t0 = time.perf_counter()
    orc.prefill(ref["cache"], st["pt"], [seq], ref["k_tscale"], ref["q_codes"], ref["q_scales"],
                ref["q_tscale"], [0, seq], [0], items)
    dt = time.perf_counter() - t0
    flops = float(sum(4 * 128 * (int(i) + 1) for i in pos))
    return {"value": flops / dt / 1e12, "unit": "TFLOP/s", "cores": orc.num_threads(),
            "kind": "oracle",
            "sample": f"{len(pos)} query rows of head 0 (positions spread over 0..{seq - 1}), "
                      f"{flops:.3e} FLOP in {dt:.2f} s; quantization not timed"}


def cpu_baseline_decode(np, W, sd):
    """Time the CPU oracle's split-KV decode on a bounded sample of the decode
    batch: the shortest and the median sequence, every query head, the batch's
    partition.  The oracle quantizes those contexts itself (statistics over the
    context, then the new token appended with them frozen), untimed; the decode
    call is timed and its algorithmic bytes counted as for the GPU launch."""
    from oracle import oracle as orc
    orc.build()
    wl = sd["wl"]
    lens = np.asarray(sd["lens"])
    order = np.argsort(lens)
    picks = [int(order[0]), int(order[len(order) // 2])]
    dt = 0.0
    nbytes = 0
    calls = []
    for b in picks:
        kv = int(lens[b])
        ctx = kv - 1
        log(f"cpu baseline: oracle quantization of decode sequence {b} ({ctx} context tokens) ...")
        q, k, v = W.gen_qkv(wl.seed, [ctx], wl.h_q, wl.h_kv, wl.outliers, "cuda", seq_ids=[b])
        npg = (kv + 63) // 64
        pt = np.arange(npg, dtype=np.int32).reshape(1, npg)
        r0 = orc.quantize_qk(W.bits(q), W.bits(k), W.bits(v), np.array([0, ctx], np.int32),
                             np.arange(ctx, dtype=np.int64), npg, orc.SMOOTH | orc.COMPUTE_STATS)
        del q, k, v
        qn, kn, vn = W.gen_qkv(wl.seed, [1], wl.h_q, wl.h_kv, wl.outliers, "cuda", tok_offsets=[ctx],
                               seq_ids=[b])
        r = orc.quantize_qk(W.bits(qn), W.bits(kn), W.bits(vn), np.array([0, 1], np.int32),
                            np.array([ctx], np.int64), npg, orc.SMOOTH, q_mean=r0["q_mean"],
                            k_mean=r0["k_mean"], k_tscale=r0["k_tscale"], cache=r0["cache"])
        items = np.array([(0, h) for h in range(wl.h_q)], np.int32)
        calls.append((r, pt, kv, items, kv * (wl.h_kv * 200 + wl.h_q * 2) + wl.h_q * (72 + 4 + 256) + npg * 4 + 4))
    # the decode calls repeated until about 10 s of CPU time have been measured
    reps = 0
    while reps == 0 or (dt < 10.0 and reps < 200):
        for r, pt, kv, items, nb in calls:
            t0 = time.perf_counter()
            orc.decode(r["cache"], pt, np.array([kv], np.int32), r["k_tscale"], r["q_codes"], r["q_scales"],
                       r["q_tscale"], sd["part"], items, smooth=True)
            dt += time.perf_counter() - t0
            nbytes += nb
        reps += 1
    return {"value": nbytes / dt / 1e9, "unit": "GB/s", "cores": orc.num_threads(), "kind": "oracle",
            "sample": f"sequences {picks} of the decode batch (contexts {[int(lens[b]) for b in picks]}), "
                      f"all {wl.h_q} query heads, partition {sd['part']}, {reps} repetitions: {nbytes:.3e} "
                      f"algorithmic bytes in {dt:.2f} s; quantization not timed"}


def softmax_ablation(torch, np, mp, W, seq, args):
    """Softmax stage costs of the prefill by the ablation chain (Sec. 3.2, Fig. 3c):
    the same launch timed with the full softmax, with P = its exponent argument
    (no exp2), and additionally without row max, row sum and O rescale.  Runs
    the characterization library libmpfa_ablate.so (outputs meaningless by
    design); the product library is restored afterwards."""
    import ctypes as C
    product = mp.LIB_PATH
    path = os.path.join(os.path.dirname(mp.LIB_PATH), "libmpfa_ablate.so")
    out = {"note": "HIP events, mean of --steps launches per level; costs are differences "
                   "between levels (exp2 = full - level 1; max/sum/rescale = level 1 - level 2)"}
    try:
        mp.LIB_PATH = path
        L = mp.lib()
        L.mpfa_ablation_set_level.restype = C.c_int
        L.mpfa_ablation_set_level.argtypes = [C.c_int]
        for name, mx in (("nvfp4", False), ("mxfp4", True)):
            log(f"softmax ablation chain, {name} ...")
            st = setup_prefill(torch, np, mp, W, seq, smooth=True, mx=mx)
            run_quant(mp, st)
            ms = []
            for level in (0, 1, 2):
                assert L.mpfa_ablation_set_level(level) == 0
                for _ in range(args.warmup):
                    run_prefill(mp, st)
                torch.cuda.synchronize()
                ts = []
                for _ in range(args.steps):
                    with Timer(torch) as t:
                        run_prefill(mp, st)
                    ts.append(t)
                ms.append(sum(t.ms() for t in ts) / args.steps)
            L.mpfa_ablation_set_level(0)
            out[name] = {"full_ms": ms[0], "no_exp2_ms": ms[1], "no_softmax_stats_ms": ms[2],
                         "exp2_ms": ms[0] - ms[1], "exp2_frac": (ms[0] - ms[1]) / ms[0],
                         "max_sum_rescale_ms": ms[1] - ms[2], "max_sum_rescale_frac": (ms[1] - ms[2]) / ms[0]}
            log(f"  {name}: full {ms[0]:.2f} ms, exp2 {ms[0] - ms[1]:.2f} ms ({100 * (ms[0] - ms[1]) / ms[0]:.1f} %), "
                f"max/sum/rescale {ms[1] - ms[2]:.2f} ms ({100 * (ms[1] - ms[2]) / ms[0]:.1f} %)")
            del st
            torch.cuda.empty_cache()
    finally:
        mp.LIB_PATH = product
    return out


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "one GPU only: the kernels run on a single MI355X; sharding heads "
                                   "or sequences across GPUs is not built"}))
        sys.exit(2)
    import torch
    import paper_2609_33135_amd as mp
    from paper_2609_33135_amd import workloads as W
    import numpy as np

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    mp.lib()
    res = {}
    prefill_ms = quant_ms = decode_ms = 0.0
    acc = {}
    seq = args.prefill_seq

    if not args.no_prefill:
        log(f"setup prefill {seq} tokens ...")
        st = setup_prefill(torch, np, mp, W, seq, smooth=True)
        for _ in range(args.warmup):
            run_quant(mp, st)
            run_prefill(mp, st)
        torch.cuda.synchronize()
        qt, pt_ = [], []
        for _ in range(args.steps):
            with Timer(torch) as t1:
                run_quant(mp, st)
            with Timer(torch) as t2:
                run_prefill(mp, st)
            qt.append(t1)
            pt_.append(t2)
        torch.cuda.synchronize()
        quant_ms = sum(t.ms() for t in qt) / args.steps
        prefill_ms = sum(t.ms() for t in pt_) / args.steps
        acc = {}
        if not args.no_accuracy:
            log("FP64 reference attention on sampled rows ...")
            ref64 = fp64_reference(np, st, 8, 24)
            acc["sample"] = (f"{len(ref64['rows'])} query rows spread over 0..{seq - 1} x "
                             f"query heads {ref64['heads']}; FP64 softmax attention of the "
                             "unquantized BF16 inputs")
            acc["nvfp4_smoothed"] = error_vs_fp64(np, st["out"], ref64)
        wl = st["wl"]
        pairs = wl.causal_pairs()
        f_qk = 2.0 * 128 * pairs
        f_pv = 2.0 * 128 * pairs
        flops = f_qk + f_pv
        achieved = flops / (prefill_ms * 1e-3)
        roof_t = f_qk / PEAK_FP4 + f_pv / PEAK_FP8
        peak = flops / roof_t
        qb = quant_bytes(wl, seq)
        res["prefill"] = {"ms": prefill_ms, "ms_min": min(t.ms() for t in pt_), "tflops": achieved / 1e12,
                          "quant_ms": quant_ms,
                          "layer_ms": quant_ms + prefill_ms,
                          "causal_pairs": pairs, "flop": flops}
        res["quant"] = {"ms": quant_ms, "bytes": qb, "GB/s": qb / (quant_ms * 1e-3) / 1e9,
                        "frac_hbm": qb / (quant_ms * 1e-3) / PEAK_HBM,
                        "kernels": "stats_partial_kernel + stats_final_kernel + quantize_kernel"}
        res["roofline"] = {"bound": "mfma", "achieved": achieved / 1e12, "peak": peak / 1e12,
                           "unit": "TFLOP/s", "frac": achieved / peak,
                           "traffic": measured_traffic("prefill_kernel"),
                           "kernel": "prefill_kernel<kSeedInit>",
                           "peak_note": "time-weighted FP4 (QK) + FP8 (PV) dense peak; exact-NVFP4 "
                                        "path peak (FP16 QK + FP8 PV) is "
                                        f"{flops / (f_qk / PEAK_BF16 + f_pv / PEAK_FP8) / 1e12:.0f}"}
        if not args.no_direct:
            log("prefill with the compensation formed by the rank-one BF16 MFMA ...")
            st["flags"] = mp.SMOOTH | mp.SEED_MFMA
            for _ in range(args.warmup):
                run_prefill(mp, st)
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t2:
                    run_prefill(mp, st)
                ts.append(t2)
            torch.cuda.synchronize()
            res["prefill"]["seed_mfma_ms"] = sum(t.ms() for t in ts) / args.steps
            log("prefill with the compensation added element-wise (placement comparison) ...")
            st["flags"] = mp.SMOOTH | mp.SEED_ELEMWISE
            for _ in range(args.warmup):
                run_prefill(mp, st)
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t2:
                    run_prefill(mp, st)
                ts.append(t2)
            torch.cuda.synchronize()
            res["prefill"]["seed_elementwise_ms"] = sum(t.ms() for t in ts) / args.steps
            st["flags"] = mp.SMOOTH
            log("prefill direct (unsmoothed) variant ...")
            del st["cache"]
            std = setup_prefill(torch, np, mp, W, seq, smooth=False)
            for _ in range(args.warmup):
                run_quant(mp, std)
                run_prefill(mp, std)
            ts, tq = [], []
            for _ in range(args.steps):
                with Timer(torch) as t1:
                    run_quant(mp, std)
                with Timer(torch) as t2:
                    run_prefill(mp, std)
                tq.append(t1)
                ts.append(t2)
            torch.cuda.synchronize()
            direct_ms = sum(t.ms() for t in ts) / args.steps
            dq_ms = sum(t.ms() for t in tq) / args.steps
            res["prefill"]["direct_quant_ms"] = dq_ms
            res["prefill"]["direct_layer_ms"] = dq_ms + direct_ms
            if acc:
                acc["nvfp4_direct"] = error_vs_fp64(np, std["out"], ref64)
            res["prefill"]["direct_ms"] = direct_ms
            res["prefill"]["rank_one_overhead"] = prefill_ms / direct_ms - 1.0
            res["prefill"]["seed_mfma_overhead"] = res["prefill"]["seed_mfma_ms"] / direct_ms - 1.0
            res["prefill"]["elementwise_overhead"] = res["prefill"]["seed_elementwise_ms"] / direct_ms - 1.0
            del std
        if not args.no_cpu_baseline:
            res["cpu_baseline"] = cpu_baseline(np, W, st, args.cpu_rows)
        del st
        torch.cuda.empty_cache()
        if not args.no_mxfp4:
            log("prefill, MXFP4 variant (E8M0 per 32, QK on the scaled FP4 MFMA) ...")
            sm = setup_prefill(torch, np, mp, W, seq, smooth=True, mx=True)
            for _ in range(args.warmup):
                run_quant(mp, sm)
                run_prefill(mp, sm)
            torch.cuda.synchronize()
            qt, ts = [], []
            for _ in range(args.steps):
                with Timer(torch) as t1:
                    run_quant(mp, sm)
                with Timer(torch) as t2:
                    run_prefill(mp, sm)
                qt.append(t1)
                ts.append(t2)
            torch.cuda.synchronize()
            mx_ms = sum(t.ms() for t in ts) / args.steps
            if acc:
                acc["mxfp4_smoothed"] = error_vs_fp64(np, sm["out"], ref64)
                sm["flags"] = mp.MXFP4
                run_quant(mp, sm)
                run_prefill(mp, sm)
                torch.cuda.synchronize()
                acc["mxfp4_direct"] = error_vs_fp64(np, sm["out"], ref64)
            mx_tf = flops / (mx_ms * 1e-3)
            mq_ms = sum(t.ms() for t in qt) / args.steps
            res["prefill_mxfp4"] = {"ms": mx_ms, "tflops": mx_tf / 1e12,
                                    "frac_fp4_fp8_peak": mx_tf / peak,
                                    "quant_ms": mq_ms, "layer_ms": mq_ms + mx_ms}
            del sm
            torch.cuda.empty_cache()

    if args.ablation:
        res["softmax_ablation"] = softmax_ablation(torch, np, mp, W, seq, args)

    if not args.no_prefill and not args.no_sweep:
        # Llama-3.1-8B-shaped prefill over the paper's range of lengths (Sec. 7.2
        # reports 16K-128K on this shape): NVFP4 (headline format) and MXFP4
        sweep = {}
        for n in (16384, 32768, 65536):
            wl_n = W.llama_prefill(n)
            f_n = 4.0 * 128 * wl_n.causal_pairs()
            row = {}
            for name, mx in (("nvfp4", False), ("mxfp4", True)):
                log(f"prefill sweep: llama shape {n} tokens, {name} ...")
                sw = setup_prefill(torch, np, mp, W, n, smooth=True, mx=mx, wl=wl_n)
                run_quant(mp, sw)
                for _ in range(max(args.warmup, 1)):
                    run_prefill(mp, sw)
                torch.cuda.synchronize()
                ts = []
                for _ in range(args.steps):
                    with Timer(torch) as t2:
                        run_prefill(mp, sw)
                    ts.append(t2)
                torch.cuda.synchronize()
                ms = sum(t.ms() for t in ts) / args.steps
                row[name] = {"ms": ms, "tflops": f_n / (ms * 1e-3) / 1e12}
                del sw
                torch.cuda.empty_cache()
            sweep[str(n)] = row
        res["prefill_llama_sweep"] = sweep

    if not args.no_prefill and not args.no_precision:
        # the other precision assignments of the PV product (Sec. 3.1, Fig. 3a)
        pa = {"nvfp4_fp8": {"ms": prefill_ms, "tflops": flops / (prefill_ms * 1e-3) / 1e12}}
        for name, pv in (("nvfp4_bf16", mp.PV_BF16), ("nvfp4_nvfp4", mp.PV_NVFP4)):
            log(f"prefill, PV precision {name} ...")
            sp = setup_prefill(torch, np, mp, W, seq, smooth=True, pv=pv)
            for _ in range(max(args.warmup, 1)):
                run_quant(mp, sp)
                run_prefill(mp, sp)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t2:
                    run_prefill(mp, sp)
                ts.append(t2)
            torch.cuda.synchronize()
            ms = sum(t.ms() for t in ts) / args.steps
            pa[name] = {"ms": ms, "tflops": flops / (ms * 1e-3) / 1e12, "time_vs_fp8": ms / prefill_ms}
            if acc:
                acc[name] = error_vs_fp64(np, sp["out"], ref64)
            del sp
            torch.cuda.empty_cache()
        res["precision_assignments"] = pa

    if acc:
        res["accuracy_vs_fp64"] = acc

    if not args.no_decode:
        log(f"setup decode batch {args.decode_batch} ...")
        sd = setup_decode(torch, np, mp, W, args.decode_batch)
        for _ in range(args.warmup):
            run_decode(mp, sd)
        torch.cuda.synchronize()
        ts = []
        for _ in range(args.steps):
            with Timer(torch) as t:
                run_decode(mp, sd)
            ts.append(t)
        torch.cuda.synchronize()
        decode_ms = sum(t.ms() for t in ts) / args.steps
        nbytes = decode_bytes(sd)
        gbs = nbytes / (decode_ms * 1e-3) / 1e9
        try:
            graph = decode_graph_replay(torch, mp, sd, args.steps, args.warmup)
        except Exception as e:   # a capture problem must not cost the benchmark line
            log(f"decode graph replay skipped: {e}")
            graph = {"error": str(e)}
        if not args.no_cpu_baseline:
            cpu_dec = cpu_baseline_decode(np, W, sd)
            res.setdefault("cpu_baseline", {"kind": "oracle"})["decode"] = cpu_dec
        res["decode"] = {"ms": decode_ms, "ms_min": min(t.ms() for t in ts), "GB/s": gbs,
                         "frac_hbm": gbs * 1e9 / PEAK_HBM,
                         "bytes": nbytes, "traffic": measured_traffic("decode_kernel"),
                         "partition_tokens": sd["part"],
                         "keys": int(sum(sd["lens"])), "graph": graph}
        del sd
        torch.cuda.empty_cache()
        if not args.no_direct:
            # the direct variant reads no Delta_S side cache (Sec. 7.2 puts that
            # cache at about 4 % of the KV bytes)
            log("decode, direct (unsmoothed) variant ...")
            sdd = setup_decode(torch, np, mp, W, args.decode_batch, smooth=False)
            for _ in range(args.warmup):
                run_decode(mp, sdd)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t:
                    run_decode(mp, sdd)
                ts.append(t)
            torch.cuda.synchronize()
            dd_ms = sum(t.ms() for t in ts) / args.steps
            dd_bytes = decode_bytes(sdd)
            res["decode"]["direct_ms"] = dd_ms
            res["decode"]["direct_GB/s"] = dd_bytes / (dd_ms * 1e-3) / 1e9
            res["decode"]["smoothing_overhead"] = decode_ms / dd_ms - 1.0
            res["decode"]["side_cache_byte_share"] = 1.0 - dd_bytes / nbytes
            del sdd
            torch.cuda.empty_cache()
        if not args.no_decode128k:
            # every context at 131072 tokens: the "128K decode" point of the target
            log("decode, batch of 131072-token contexts ...")
            s128 = setup_decode(torch, np, mp, W, args.decode_batch, ctx_range=(131072, 131072))
            for _ in range(args.warmup):
                run_decode(mp, s128)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t:
                    run_decode(mp, s128)
                ts.append(t)
            torch.cuda.synchronize()
            d128_ms = sum(t.ms() for t in ts) / args.steps
            d128_bytes = decode_bytes(s128)
            res["decode_128k"] = {"ms": d128_ms, "GB/s": d128_bytes / (d128_ms * 1e-3) / 1e9,
                                  "frac_hbm": d128_bytes / (d128_ms * 1e-3) / PEAK_HBM,
                                  "bytes": d128_bytes, "partition_tokens": s128["part"],
                                  "contexts": f"{args.decode_batch} x 131072"}
            del s128
            torch.cuda.empty_cache()
        if not args.no_mxfp4:
            log("decode, MXFP4 variant ...")
            sx = setup_decode(torch, np, mp, W, args.decode_batch, mx=True)
            for _ in range(args.warmup):
                run_decode(mp, sx)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t:
                    run_decode(mp, sx)
                ts.append(t)
            torch.cuda.synchronize()
            mx_ms = sum(t.ms() for t in ts) / args.steps
            mx_bytes = decode_bytes(sx)
            res["decode_mxfp4"] = {"ms": mx_ms, "GB/s": mx_bytes / (mx_ms * 1e-3) / 1e9,
                                   "frac_hbm": mx_bytes / (mx_ms * 1e-3) / PEAK_HBM,
                                   "bytes": mx_bytes}
            del sx

    if not args.no_mixed:
        log("mixed serving step: setup ...")
        mx = setup_mixed(torch, np, mp, W)
        res_m = {}
        for name, fn in (("separate_ms", run_mixed_separate), ("fused_ms", run_mixed_fused),
                         ("fused_with_quant_ms", run_mixed_with_quant)):
            for _ in range(max(args.warmup, 1)):
                fn(mp, mx)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.steps):
                with Timer(torch) as t:
                    fn(mp, mx)
                ts.append(t)
            torch.cuda.synchronize()
            res_m[name] = sum(t.ms() for t in ts) / args.steps
        res_m["workload"] = ("qwen3-14b-shaped: 32768-token chunk at position 65536 + 64 decode sequences, "
                             f"contexts U[8192,131072] ({mx['keys']} keys, partition {mx['part']})")
        res_m["attention_tflops_fused"] = 4.0 * 128 * mx["pairs"] / (res_m["fused_ms"] * 1e-3) / 1e12
        res["mixed_step"] = res_m
        del mx
        torch.cuda.empty_cache()

    if not args.no_peaks:
        log("achievable GEMM and copy rates ...")
        pk = measured_peaks(torch)
        res["measured_peaks"] = pk
        if "prefill" in res and pk.get("fp16_gemm_tflops") and pk.get("fp8_gemm_tflops"):
            # time-weighted over the two contractions of the exact-NVFP4 path
            fl = res["prefill"]["flop"]
            t_meas = (fl / 2) / (pk["fp16_gemm_tflops"] * 1e12) + (fl / 2) / (pk["fp8_gemm_tflops"] * 1e12)
            res["roofline"]["frac_of_library_gemm"] = res["prefill"]["tflops"] * 1e12 / (fl / t_meas)
        if "decode" in res and pk.get("copy_GBps"):
            res["decode"]["frac_of_device_copy"] = res["decode"]["GB/s"] / pk["copy_GBps"]
        log("probe kernels: MFMA issue rates and HBM read rate ...")
        from paper_2609_33135_amd import probe as probe_lib
        pp = probe_peaks(torch, probe_lib)
        res["measured_peaks"]["probe"] = pp
        if "prefill" in res:
            # the same time weighting as the specification peaks: half the FLOP in
            # each contraction
            hm = lambda a, b: 2.0 / (1.0 / a + 1.0 / b)
            meas_fp4_fp8 = hm(pp["mfma_fp4_tflops"], pp["mfma_fp8_tflops"])
            meas_f16_fp8 = hm(pp["mfma_f16_tflops"], pp["mfma_fp8_tflops"])
            res["roofline"]["measured_peak"] = meas_fp4_fp8
            res["roofline"]["frac_of_measured_peak"] = res["prefill"]["tflops"] / meas_fp4_fp8
            res["roofline"]["measured_exact_path_peak"] = meas_f16_fp8
            res["roofline"]["frac_of_measured_exact_path_peak"] = res["prefill"]["tflops"] / meas_f16_fp8
        if "decode" in res:
            read = max(pp["read_vgpr_GBps"], pp["read_lds_GBps"])
            res["decode"]["frac_of_measured_read"] = res["decode"]["GB/s"] / read
        if "decode_128k" in res:
            res["decode_128k"]["frac_of_measured_read"] = res["decode_128k"]["GB/s"] / max(
                pp["read_vgpr_GBps"], pp["read_lds_GBps"])

    if args.copy_calibration:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        res["copy_calibration_bytes"] = 1 << 30

    line = {
        "metric": "prefill attn TFLOPS (causal 128K) + decode KV GB/s, % of roofline, 1 MI355X",
        "value": res.get("prefill", {}).get("tflops"),
        "unit": "TFLOP/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": quant_ms + prefill_ms + decode_ms,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "nvfp4 via exact f16 mfma (QK) + fp8 mfma (PV), f32 softmax",
        "data": "synthetic (seeded counter-based normal, per-channel K offsets, 0.1% x20 outliers)",
        "config": {"workload": f"qwen3-14b-shaped causal prefill {seq} tokens 40q/8kv d128 + "
                               f"llama-3.1-8b-shaped paged decode batch {args.decode_batch} "
                               "contexts U[16384,131072] 32q/8kv d128",
                   "prefill_seq": seq, "decode_batch": args.decode_batch, "page_tokens": 64,
                   "smoothing": True},
    }
    line.update({k: v for k, v in res.items()})
    print(json.dumps(line))


if __name__ == "__main__":
    main()
