"""Benchmark of the RRQ hot path on one MI355X.

One step = the whole path over the workload, each kernel as one flat call over
the full weight stack with every buffer resident in HBM:
  rrq_construct    (bf16 weights -> 4-stage package, G = 128)
  rrq_reconstruct  at every prefix the workload names (bf16 output).

Default workload: the 36-layer Qwen3-8B-shaped stack (6.95e9 weights,
13.9 GB bf16; Gaussian with 0.1% x20 outliers).

After the steps: rrq_construct_from_base (the residual stages on a given base
checkpoint; here the package's own stage 0) is timed on the same workload,
the per-group peak-to-mean ratio (alone, and as a side output of
construction) is timed and its tensor-level indicators reported,
construction in other stage formats (symmetric with fp16 scales, real
zero-points, bf16 scales) is timed, rrq_linear decode passes (1 and 16
tokens, prefixes k = 1..4, one call per tensor on per-tensor packages, and
with q/k/v and gate/up fused into one call each; the pass replayed as a HIP
graph and also launched call by call) are timed, and a streaming probe with the same read/write mix gives the practical HBM
ceiling (include/hbm_probe.h).

Prints one JSON line. ``value`` is construction throughput in GB/s of bf16
weights (2 bytes x weights / mean construct kernel time). The roofline entry
is for the construct kernel: algorithmic HBM bytes per launch (bf16 in,
codes + fp32 scales and zeros out) / its mean duration, against 8 TB/s.
"""

from __future__ import annotations

import argparse
import gc
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
TRAFFIC_PROFILE = os.path.join(ROOT, "profiles", "construct_kernel_g128_qwen3_8b_stack36_traffic.md")
METRIC = "RRQ 4-stage construction GB/s of bf16 weights (% HBM peak); reconstruct GB/s"


def construct_bytes(n, G, S):
    """Algorithmic HBM bytes of one construct launch: bf16 in, 2-bit codes,
    fp32 scale and zero per group and stage."""
    return 2 * n + S * n // 4 + 2 * 4 * S * (n // G)


def reconstruct_bytes(n, G, k, out_bytes):
    return k * n // 4 + 2 * 4 * k * (n // G) + out_bytes * n


def cpu_model():
    """The host CPU's model name (Linux), or None."""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def cpu_baseline(w, W_dev, budget_s=12.0, threads=0):
    """The C oracle (as it stands) on the host cores: whole tensors of the
    workload in order, passes repeated, until about budget_s seconds of
    compute (at most 64 passes). threads > 0 sets the OpenMP thread count."""
    import numpy as np
    import torch

    import oracle

    G, S = w.group_size, w.n_stages
    if threads > 0:
        oracle.c_set_threads(threads)
    threads = oracle.c_threads()
    done_elems, elapsed, n_calls, passes = 0, 0.0, 0, 0
    host = {}
    while elapsed < budget_s and passes < 64:
        for t in w.tensors:
            if t.name not in host:
                host[t.name] = (W_dev[t.offset:t.offset + t.numel].cpu().view(torch.int16)
                                .numpy().view(np.uint16))
                if len(host) > 16:   # bound host memory on large stacks
                    host.pop(next(iter(host)))
            bits = host.get(t.name)
            if bits is None:
                bits = (W_dev[t.offset:t.offset + t.numel].cpu().view(torch.int16).numpy()
                        .view(np.uint16))
            t0 = time.perf_counter()
            oracle.c_construct(bits, G, S)
            elapsed += time.perf_counter() - t0
            done_elems += t.numel
            n_calls += 1
            if elapsed >= budget_s:
                break
        passes += 1
    sample = (f"{n_calls} tensor calls over {len(w.tensors)} tensors of {w.name} "
              f"({passes} pass(es)), {done_elems} weights, construct only, {elapsed:.1f} s")
    result = {"value": round(2 * done_elems / elapsed / 1e9, 4), "unit": "GB/s", "cores": threads,
              "kind": "oracle", "sample": sample, "cpu": cpu_model()}

    # Per-core figure: one OpenMP thread on one decoder layer (the first
    # layer of a stack, i.e. the single-layer workload's bits), one pass.
    layer = [t for t in w.tensors if t.name.startswith("layers.0.")] or list(w.tensors)
    oracle.c_set_threads(1)
    try:
        el1, n1 = 0.0, 0
        for t in layer:
            bits = W_dev[t.offset:t.offset + t.numel].cpu().view(torch.int16).numpy().view(np.uint16)
            t0 = time.perf_counter()
            oracle.c_construct(bits, G, S)
            el1 += time.perf_counter() - t0
            n1 += t.numel
    finally:
        oracle.c_set_threads(threads)
    result["one_thread"] = {
        "value": round(2 * n1 / el1 / 1e9, 4), "unit": "GB/s", "cores": 1,
        "sample": f"{len(layer)} tensors of one decoder layer ({n1} weights), construct only, "
                  f"{el1:.1f} s"}
    return result


def from_base_bytes(n, G, S):
    """Algorithmic HBM bytes of one rrq_construct_from_base launch: bf16 in,
    the base stage's codes, scales and zeros in, S - 1 residual stages out."""
    return 2 * n + n // 4 + 8 * (n // G) + (S - 1) * n // 4 + 8 * (S - 1) * (n // G)


def time_from_base(calls, G, S, stream, flush_buf=None, launches=20):
    """Mean / min time of rrq_construct_from_base over the workload, with the
    package's own stage 0 (already in plane 0) as the base checkpoint."""
    import torch

    import paper_2608_04048_amd as rrq

    def run():
        for Wc, r_, c_, cc, sc, zz, _ in calls:
            rrq.rrq_construct_from_base(Wc, r_, c_, G, S, cc, sc, zz, stream)

    run()
    ms = []
    for _ in range(launches):
        if flush_buf is not None:
            flush_buf.fill_(1.0)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        run()
        b.record(stream)
        b.synchronize()
        ms.append(a.elapsed_time(b))
    return sum(ms) / len(ms), min(ms)


def decode_calls(w, fused):
    """The rrq_linear calls of one decode pass over w: one per tensor, or
    with the projections that read the same input (q/k/v, gate/up: adjacent
    in the flat buffer, same input width) fused into one call on their
    row-concatenated weight. Returns (name, rows, cols, offset) tuples."""
    calls = []
    for t in w.tensors:
        short = t.name.split(".")[-1]
        if fused and calls and short in ("k_proj", "v_proj", "up_proj"):
            name, rows, cols, off = calls[-1]
            assert cols == t.cols and off + rows * cols == t.offset
            calls[-1] = (name + "+" + short, rows + t.rows, cols, off)
        else:
            calls.append((short, t.rows, t.cols, t.offset))
    return calls


def linear_bytes(calls, G, k, M):
    """Algorithmic HBM bytes of one decode pass of rrq_linear calls: k code
    planes + k (s, z) per group, X in, Y out."""
    total = 0
    for _, rows, cols, _ in calls:
        n = rows * cols
        total += k * n // 4 + 8 * k * (n // G) + 2 * M * cols + 4 * M * rows
    return total


def time_linear(w, W_flat, codes, scales, zeros, stream, tokens=(1, 16), ks=(1, 2, 3, 4),
                launches=10):
    """Decode-style passes of rrq_linear over every tensor of w, each call on
    its own package: one call per tensor ("per_tensor"), and with q/k/v and
    gate/up fused into one call each on their row-concatenated weight
    ("fused": the same groups, so the same package bytes). A pass is
    captured once in a HIP graph and replayed, as a serving loop would run
    it, and timed with HIP events around each replay ("ms"); the same pass
    launched call by call from Python is timed too ("ms_eager"). Builds the
    packages first (untimed)."""
    import torch

    import paper_2608_04048_amd as rrq

    G, S = w.group_size, w.n_stages
    cflat, sflat, zflat = codes.view(-1), scales.view(-1), zeros.view(-1)
    g = torch.Generator(device="cuda")
    g.manual_seed(2608)
    max_m = max(tokens)
    xs = {c: torch.randn((max_m, c), generator=g, device="cuda").to(torch.bfloat16)
          for c in sorted({t.cols for t in w.tensors})}
    y = torch.empty(max_m * 2 * max(t.rows for t in w.tensors), dtype=torch.float32,
                    device="cuda")

    def timed(fn):
        fn()
        ms = []
        for _ in range(launches):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            fn()
            b.record(stream)
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return sum(ms) / len(ms)

    out = {}
    cs = torch.cuda.Stream()
    for mode in ("per_tensor", "fused"):
        calls = decode_calls(w, mode == "fused")
        pk = []
        for name, rows, cols, off in calls:
            n = rows * cols
            c = cflat[S * off // 16:S * (off + n) // 16].view(S, n // 16)
            sc = sflat[S * off // G:S * (off + n) // G].view(S, n // G)
            zz = zflat[S * off // G:S * (off + n) // G].view(S, n // G)
            rrq.rrq_construct(W_flat[off:off + n], rows, cols, G, S, c, sc, zz, stream)
            pk.append((rows, cols, c, sc, zz))
        torch.cuda.synchronize()
        res = {}
        for M in tokens:
            for k in ks:
                def run(st, M=M, k=k):
                    for rows, cols, c, sc, zz in pk:
                        rrq.rrq_linear(c, sc, zz, rows, cols, G, S, k, xs[cols], M, y, st)
                t_eager = timed(lambda: run(stream))
                cs.wait_stream(stream)
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=cs):
                    run(cs)
                stream.wait_stream(cs)

                def replay():
                    with torch.cuda.stream(stream):
                        graph.replay()
                t_ms = timed(replay)
                del graph
                nbytes = linear_bytes(calls, G, k, M)
                res[f"M{M}_k{k}"] = {"ms": round(t_ms, 4), "ms_eager": round(t_eager, 4),
                                     "bytes": nbytes,
                                     "hbm_gbs": round(nbytes / (t_ms * 1e-3) / 1e9, 1),
                                     "hbm_frac": round(nbytes / (t_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}
        res["calls"] = (f"{len(calls)} rrq_linear calls per pass "
                        f"({', '.join(sorted({c[0] for c in calls}))}), replayed as one HIP graph")
        out[mode] = res
    return out


def time_linear_shape(rows, cols, ks, tokens, G=128, S=4, min_bytes=600 << 20, replays=7):
    """rrq_linear on one weight shape, as a decode loop meets it: P distinct
    packages (seeded Gaussian weights, together at least min_bytes, so that
    every call reads its package from HBM rather than the 256 MB MALL), one
    call per package captured in a HIP graph; the graph is replayed and timed
    with HIP events. Returns per-call microseconds and algorithmic HBM
    bytes per call for every (tokens, k)."""
    import torch

    import paper_2608_04048_amd as rrq

    n = rows * cols
    P = max(2, min(64, min_bytes // (S * n // 4 + 8 * S * n // G) + 1))
    g = torch.Generator(device="cuda")
    g.manual_seed(2608)
    W = (torch.randn(n, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    stream = torch.cuda.current_stream()
    pks = []
    for _ in range(P):
        c = torch.empty((S, n // 16), dtype=torch.int32, device="cuda")
        sc = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
        zz = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
        rrq.rrq_construct(W, rows, cols, G, S, c, sc, zz, stream)
        pks.append((c, sc, zz))
    max_m = max(tokens)
    X = torch.randn((max_m, cols), generator=g, device="cuda").to(torch.bfloat16)
    Y = torch.empty((P, max_m * rows), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    out = {"metric": "rrq_linear per-call time", "rows": rows, "cols": cols, "group_size": G,
           "packages": P, "results": {}}
    cs = torch.cuda.Stream()
    for M in tokens:
        for k in ks:
            def run(st, M=M, k=k):
                for j, (c, sc, zz) in enumerate(pks):
                    rrq.rrq_linear(c, sc, zz, rows, cols, G, S, k, X, M, Y[j], st)
            run(stream)
            cs.wait_stream(stream)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=cs):
                run(cs)
            stream.wait_stream(cs)
            ms = []
            for _ in range(replays):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record(stream)
                with torch.cuda.stream(stream):
                    graph.replay()
                b.record(stream)
                b.synchronize()
                ms.append(a.elapsed_time(b))
            del graph
            us = sorted(ms)[len(ms) // 2] * 1e3 / P
            nbytes = k * n // 4 + 8 * k * (n // G) + 2 * M * cols + 4 * M * rows
            out["results"][f"M{M}_k{k}"] = {
                "us_per_call": round(us, 2), "bytes_per_call": nbytes,
                "hbm_gbs": round(nbytes / (us * 1e-6) / 1e9, 1),
                "hbm_frac": round(nbytes / (us * 1e-6) / 1e9 / HBM_PEAK_GBS, 4)}
    return out


MFMA_BF16_PEAK_TFLOPS = 2500.0


def time_prefill(tokens=2048, ks=(4, 1),
                 shapes=((4096, 4096, "q_proj/o_proj"), (12288, 4096, "gate_proj/up_proj"),
                         (4096, 12288, "down_proj"))):
    """rrq_linear at prefill size on the Qwen3-8B layer shapes (time_linear_shape):
    the product's 2 M rows cols flops (product_tflops), and the share of the bf16
    matrix-core peak of the passes that are run (mfma_frac): one per stage at 1
    and 2 stages, the split form's three at 3 and 4."""
    out = {"tokens": tokens}
    for rows, cols, name in shapes:
        r = time_linear_shape(rows, cols, list(ks), [tokens])
        for key, v in r["results"].items():
            k = int(key.split("_k")[1])
            tf = 2.0 * tokens * rows * cols / (v["us_per_call"] * 1e-6) / 1e12
            out[f"{rows}x{cols}_k{k}"] = {"proj": name, "us_per_call": v["us_per_call"],
                                          "product_tflops": round(tf, 1),
                                          "mfma_frac": round(tf * min(k, 3) / MFMA_BF16_PEAK_TFLOPS, 4)}
    return out


def format_bytes(n, G, S, zero_point, scale_type):
    """Algorithmic HBM bytes of one construct launch in a stage format:
    bf16 in, codes, scales (4 or 2 bytes) and zeros (none if symmetric)."""
    sb = 4 if scale_type == "f32" else 2
    zb = 0 if zero_point == "sym" else 4
    return 2 * n + S * n // 4 + (sb + zb) * S * (n // G)


def time_formats(W, n, G, S, stream, formats=(("sym", "f16"), ("real", "f32"), ("int", "bf16")),
                 launches=10):
    """Mean time of rrq_construct_format over the flat workload per format."""
    import torch

    import paper_2608_04048_amd as rrq

    rows, cols = W.shape
    codes = torch.empty((S, n // 16), dtype=torch.int32, device="cuda")
    zeros = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
    out = {}
    for zp, sd in formats:
        scales = torch.empty((S, n // G), dtype=torch.float32 if sd == "f32" else torch.int16,
                             device="cuda")

        def run():
            rrq.rrq_construct_format(W, rows, cols, G, S, rrq.ZERO_POINTS[zp], rrq.SCALE_TYPES[sd],
                                     codes, scales, None if zp == "sym" else zeros, stream)
        run()
        ms = []
        for _ in range(launches):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            run()
            b.record(stream)
            b.synchronize()
            ms.append(a.elapsed_time(b))
        t = sum(ms) / len(ms)
        nb = format_bytes(n, G, S, zp, sd)
        out[f"{zp}_{sd}"] = {"ms": round(t, 4), "gbs_bf16_weights": round(2 * n / (t * 1e-3) / 1e9, 1),
                             "hbm_gbs": round(nb / (t * 1e-3) / 1e9, 1),
                             "hbm_frac": round(nb / (t * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                             "bytes_per_launch": nb}
        del scales
    del codes, zeros
    return out


def time_pmr(w, W, G, S, stream, launches=10):
    """rrq_group_pmr over the flat workload (HBM: 2 bytes in, 4/G out per
    weight), rrq_construct_stats against plain construction, and the paper's
    tensor-level outlier indicators (mean and maximum over tensors of the
    largest group PMR of each tensor) for the workload."""
    import torch

    import paper_2608_04048_amd as rrq

    rows, cols = W.shape
    n = rows * cols
    pmr = torch.empty(n // G, dtype=torch.float32, device="cuda")
    codes = torch.empty((S, n // 16), dtype=torch.int32, device="cuda")
    scales = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
    zeros = torch.empty((S, n // G), dtype=torch.float32, device="cuda")

    def timed(fn):
        fn()
        ms = []
        for _ in range(launches):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            fn()
            b.record(stream)
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return sum(ms) / len(ms)

    t_pmr = timed(lambda: rrq.rrq_group_pmr(W, rows, cols, G, pmr, stream))
    t_stats = timed(lambda: rrq.rrq_construct_stats(W, rows, cols, G, S, rrq.RRQ_ZP_INTEGER,
                                                    rrq.RRQ_SCALE_F32, codes, scales, zeros,
                                                    pmr, stream))
    t_plain = timed(lambda: rrq.rrq_construct(W, rows, cols, G, S, codes, scales, zeros, stream))
    tmax = [float(pmr[t.offset // G:(t.offset + t.numel) // G].max()) for t in w.tensors]
    pbytes = 2 * n + 4 * (n // G)
    del codes, scales, zeros, pmr
    return {"group_pmr_ms": round(t_pmr, 4), "group_pmr_hbm_gbs": round(pbytes / (t_pmr * 1e-3) / 1e9, 1),
            "group_pmr_hbm_frac": round(pbytes / (t_pmr * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
            "construct_stats_ms": round(t_stats, 4), "construct_ms_same_run": round(t_plain, 4),
            "mean_tensor_max_pmr": round(sum(tmax) / len(tmax), 3),
            "max_tensor_max_pmr": round(max(tmax), 3)}


def stream_probe(src_bytes, flush_buf=None, launches=10):
    """Practical HBM ceiling for construction's read/write mix: a streaming
    kernel reading src_bytes and writing 5/8 of that (include/hbm_probe.h),
    mean of `launches` HIP-event-timed launches on the current stream; and the
    read-only and write-only probes on the same byte counts."""
    import torch

    from paper_2608_04048_amd import probe

    src_bytes -= src_bytes % 128
    src = torch.empty(src_bytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
    dst = torch.empty(src_bytes // 8 * 5 // 4, dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream()
    for _ in range(2):
        probe.hbm_probe_stream(src, src_bytes, dst, stream)
    ms = []
    for _ in range(launches):
        if flush_buf is not None:
            flush_buf.fill_(1.0)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        probe.hbm_probe_stream(src, src_bytes, dst, stream)
        b.record(stream)
        b.synchronize()
        ms.append(a.elapsed_time(b))
    t = sum(ms) / len(ms)
    moved = src_bytes + src_bytes // 8 * 5
    gbs = moved / (t * 1e-3) / 1e9

    # Each direction alone: the read-only probe on src, the write-only probe
    # on dst (the same byte counts). "serial" is the rate of reading and then
    # writing those bytes one after the other at these rates.
    out = torch.zeros(1, dtype=torch.int32, device="cuda")

    def timed(fn):
        fn()
        vals = []
        for _ in range(launches):
            if flush_buf is not None:
                flush_buf.fill_(1.0)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            fn()
            b.record(stream)
            b.synchronize()
            vals.append(a.elapsed_time(b))
        return sum(vals) / len(vals)

    t_read = timed(lambda: probe.hbm_probe_read(src, src_bytes, out, stream))
    t_write = timed(lambda: probe.hbm_probe_write(dst, src_bytes // 8 * 5, 0, stream))
    del src, dst
    read_gbs = src_bytes / (t_read * 1e-3) / 1e9
    write_gbs = src_bytes // 8 * 5 / (t_write * 1e-3) / 1e9
    serial_gbs = moved / ((t_read + t_write) * 1e-3) / 1e9
    return {"read_bytes": src_bytes, "written_bytes": src_bytes // 8 * 5, "ms": round(t, 4),
            "gbs": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4),
            "read_only": {"ms": round(t_read, 4), "gbs": round(read_gbs, 1),
                          "frac": round(read_gbs / HBM_PEAK_GBS, 4)},
            "write_only": {"ms": round(t_write, 4), "gbs": round(write_gbs, 1),
                           "frac": round(write_gbs / HBM_PEAK_GBS, 4)},
            "serial": {"ms": round(t_read + t_write, 4), "gbs": round(serial_gbs, 1),
                       "frac": round(serial_gbs / HBM_PEAK_GBS, 4)}}


def machine_probe(iters_issue=20000, iters_lds=4000):
    """The machine terms the linear-layer kernels are built from, from the
    probes of libhbm_probe.so (hbm_probe_issue, hbm_probe_lds): s_memtime
    ticks per wave of a loop of v_mfma_f32_16x16x32_bf16 (16 per iteration,
    4 chains), of binary32 FMAs (64, 8 chains) and of both interleaved, at 1,
    2 and 4 waves per SIMD; and of 16-byte LDS reads at 4 and 8 waves per
    compute unit. Second of two launches each."""
    import torch

    from paper_2608_04048_amd import probe

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    res = {"issue": {}, "lds": {}}
    for wps in (1, 2, 4):
        out = torch.empty(cus * wps * 256, dtype=torch.float32, device="cuda")
        ticks = torch.empty(cus * wps * 4, dtype=torch.int64, device="cuda")
        per = {}
        for mode, name in ((0, "mfma16"), (1, "fma64"), (2, "mfma16_fma64")):
            for _ in range(2):
                probe.hbm_probe_issue(mode, wps, iters_issue, out, ticks)
            torch.cuda.synchronize()
            per[name] = ticks.double().mean().item() / iters_issue
        res["issue"][str(wps)] = {
            "ticks_per_iter_per_wave": {k: round(v, 1) for k, v in per.items()},
            "ticks_per_mfma_per_simd": round(per["mfma16"] / 16 / wps, 2),
            "ticks_per_fma_per_simd": round(per["fma64"] / 64 / wps, 2),
            "both_over_mfma": round(per["mfma16_fma64"] / per["mfma16"], 3),
            "both_over_sum": round(per["mfma16_fma64"] / (per["mfma16"] + per["fma64"]), 3),
        }
    for wpc in (4, 8):
        out = torch.empty(cus * wpc * 64, dtype=torch.int32, device="cuda")
        ticks = torch.empty(cus * wpc, dtype=torch.int64, device="cuda")
        for _ in range(2):
            probe.hbm_probe_lds(wpc, iters_lds, out, ticks)
        torch.cuda.synchronize()
        t = ticks.double().mean().item()
        reads = iters_lds * 16 * wpc                      # per compute unit
        res["lds"][str(wpc)] = {"ticks_per_read_per_cu": round(t / reads, 2),
                                "bytes_per_tick_per_cu": round(reads * 1024 / t, 1)}
    return res


def time_per_tensor(w, W_flat, codes, scales, zeros, stream, passes=5, n_streams=4):
    """Each weight tensor into its own package (laid out back to back in the
    package buffers), the way a checkpoint stored tensor by tensor is
    quantized: one rrq_construct call per tensor issued from Python on one
    stream; the same calls spread round-robin over n_streams streams and
    captured once in a HIP graph (the tensors are independent, so one
    call's last waves overlap the next calls' first ones, and the host's
    per-call launch cost leaves the timed pass); and every tensor in one
    rrq_construct_many call. Mean time of one pass over every tensor, HIP
    events on the launch stream; the graph's packages are checked equal to
    the eager calls'."""
    import torch

    import paper_2608_04048_amd as rrq

    G, S, n = w.group_size, w.n_stages, w.numel
    cflat, sflat, zflat = codes.view(-1), scales.view(-1), zeros.view(-1)
    calls = []
    for t in w.tensors:
        c = cflat[S * t.offset // 16:S * (t.offset + t.numel) // 16].view(S, t.numel // 16)
        sc = sflat[S * t.offset // G:S * (t.offset + t.numel) // G].view(S, t.numel // G)
        zz = zflat[S * t.offset // G:S * (t.offset + t.numel) // G].view(S, t.numel // G)
        calls.append((W_flat[t.offset:t.offset + t.numel], t.rows, t.cols, c, sc, zz))

    def one_pass():
        for Wc, r_, c_, cc, sc, zz in calls:
            rrq.rrq_construct(Wc, r_, c_, G, S, cc, sc, zz, stream)

    def many():
        rrq.rrq_construct_many(calls, G, S, stream)

    def package_sum():
        return (int(codes.sum(dtype=torch.int64)), float(scales.sum(dtype=torch.float64)),
                float(zeros.sum(dtype=torch.float64)))

    # the per-tensor calls on n_streams streams, captured once (default
    # priority streams; the capture stream forks to them and joins back)
    cap = torch.cuda.Stream()
    side = [torch.cuda.Stream() for _ in range(n_streams)]
    one_pass()
    torch.cuda.synchronize()
    eager_sum = package_sum()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        fork = torch.cuda.Event()
        fork.record(cap)
        for sd in side:
            sd.wait_event(fork)
        for i, (Wc, r_, c_, cc, sc, zz) in enumerate(calls):
            rrq.rrq_construct(Wc, r_, c_, G, S, cc, sc, zz, side[i % n_streams])
        for sd in side:
            join = torch.cuda.Event()
            join.record(sd)
            cap.wait_event(join)

    def graphed():
        graph.replay()

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        gc.collect()
        gc.disable()   # a collection pause would let the queue drain mid-pass
        ms = []
        for _ in range(passes):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            fn()
            b.record(stream)
            b.synchronize()
            ms.append(a.elapsed_time(b))
        gc.enable()
        return sum(ms) / len(ms)

    cb = construct_bytes(n, G, S)
    out = {}
    for key, fn, ncalls in (("calls", one_pass, len(calls)), ("calls_graph", graphed, len(calls)),
                            ("one_call", many, 1)):
        t = timed(fn)
        if key == "calls_graph":
            torch.cuda.synchronize()
            if package_sum() != eager_sum:
                raise RuntimeError("bench: the graph-replayed per-tensor packages differ "
                                   "from the eager calls'")
        out[key] = {"api": "rrq_construct_many" if key == "one_call" else "rrq_construct",
                    "calls": ncalls, "construct_ms": round(t, 4),
                    "gbs_bf16_weights": round(2 * n / (t * 1e-3) / 1e9, 1),
                    "hbm_gbs": round(cb / (t * 1e-3) / 1e9, 1),
                    "hbm_frac": round(cb / (t * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}
    out["calls_graph"]["streams"] = n_streams
    out["calls_graph"]["launch"] = "one HIP graph per pass, calls round-robin over the streams"
    out["tensors"] = len(calls)
    del graph
    return out


def construct_probe(W, n, G, S, codes, scales, zeros, stream, flush_buf=None, launches=10,
                    blocks_per_cu=(8, 4, 16)):
    """Construction's own memory traffic with no arithmetic
    (hbm_probe_construct): the same input, the same output planes and
    addresses as the construct call, the same tiles and launch (8 one-wave
    workgroups per CU), and the same workload; also at other occupancies.
    Overwrites the package buffers."""
    import torch

    from paper_2608_04048_amd import probe

    moved = construct_bytes(n, G, S)
    out = {}
    for bpc in blocks_per_cu:
        def run():
            probe.hbm_probe_construct(W, n // G, G, S, codes, scales, zeros, bpc, stream)
        run()
        vals = []
        for _ in range(launches):
            if flush_buf is not None:
                flush_buf.fill_(1.0)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            run()
            b.record(stream)
            b.synchronize()
            vals.append(a.elapsed_time(b))
        t = sum(vals) / len(vals)
        gbs = moved / (t * 1e-3) / 1e9
        out[bpc] = {"ms": round(t, 4), "gbs": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4)}
    res = dict(out[blocks_per_cu[0]])
    res["bytes"] = moved
    res["by_blocks_per_cu"] = {str(k): v for k, v in out.items()}
    return res


def reconstruct_probe(n, G, ks, codes, scales, zeros, outs, stream, flush_buf=None,
                      launches=10):
    """Reconstruction's memory traffic with no arithmetic
    (hbm_probe_reconstruct), bfloat16 out, at every prefix k the workload
    reconstructs: the same package planes and output buffers and the same
    launch as rrq_reconstruct (two 256-thread workgroups per CU)."""
    import torch

    from paper_2608_04048_amd import probe

    res = {}
    for k in ks:
        def run():
            probe.hbm_probe_reconstruct(codes, scales, zeros, n // G, G, k, outs[k], 0, stream)
        run()
        vals = []
        for _ in range(launches):
            if flush_buf is not None:
                flush_buf.fill_(1.0)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            run()
            b.record(stream)
            b.synchronize()
            vals.append(a.elapsed_time(b))
        t = sum(vals) / len(vals)
        moved = reconstruct_bytes(n, G, k, 2)
        gbs = moved / (t * 1e-3) / 1e9
        res[str(k)] = {"ms": round(t, 4), "gbs": round(gbs, 1),
                       "frac": round(gbs / HBM_PEAK_GBS, 4), "bytes": moved}
    return res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="qwen3_8b_stack36")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--per-tensor", action="store_true",
                    help="one construct / reconstruct call per weight tensor (each tensor its "
                         "own package) instead of one flat call over the whole stack")
    ap.add_argument("--cpu-budget", type=float, default=12.0, metavar="S",
                    help="seconds of oracle compute for the CPU baseline sample")
    ap.add_argument("--cpu-threads", type=int, default=0, metavar="N",
                    help="OpenMP threads for the CPU baseline (default: all the runtime gives)")
    ap.add_argument("--flush-mall", choices=("auto", "on", "off"), default="auto",
                    help="write a 512 MiB buffer before each step so no input starts in the "
                         "256 MB MALL (auto: on when the step moves under 4 GB)")
    ap.add_argument("--no-from-base", action="store_true",
                    help="skip timing rrq_construct_from_base (residual stages on a given base)")
    ap.add_argument("--no-pmr", action="store_true",
                    help="skip timing the peak-to-mean ratio side output")
    ap.add_argument("--no-formats", action="store_true",
                    help="skip timing rrq_construct_format in other stage formats")
    ap.add_argument("--no-linear", action="store_true",
                    help="skip timing rrq_linear (decode passes over every tensor)")
    ap.add_argument("--no-stream-probe", action="store_true",
                    help="skip the 2 : 1.25 read/write streaming probe")
    ap.add_argument("--linear-shape", default="", metavar="RxC",
                    help="instead of the benchmark, time rrq_linear on one weight shape: one "
                         "call per package over enough distinct packages to exceed the 256 MB "
                         "MALL, replayed as a HIP graph (per-call microseconds)")
    ap.add_argument("--linear-k", default="4", metavar="K,...",
                    help="prefix stage counts for --linear-shape")
    ap.add_argument("--linear-tokens", default="1", metavar="M,...",
                    help="token counts for --linear-shape")
    ap.add_argument("--machine-probe", action="store_true",
                    help="print the instruction-issue and LDS-read probes' figures and exit")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="instead of the benchmark, run a plain device-to-device copy of MIB "
                         "MiB three times (calibrates profiler byte counters)")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: the benchmark runs on one GPU only (the path needs no exchange between "
              "GPUs); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2608_04048_amd as rrq
    from paper_2608_04048_amd import workloads as wl

    torch.cuda.set_device(0)
    if args.machine_probe:
        print(json.dumps({"machine_probe": machine_probe()}), flush=True)
        return
    if args.copy_probe:
        src = torch.ones(args.copy_probe << 18, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes": src.numel() * 4, "copies": 3}), flush=True)
        return
    rrq.load_library()
    if args.linear_shape:
        rows, cols = (int(v) for v in args.linear_shape.lower().split("x"))
        print(json.dumps(time_linear_shape(rows, cols, [int(k) for k in args.linear_k.split(",")],
                                           [int(m) for m in args.linear_tokens.split(",")])),
              flush=True)
        return
    w = wl.workload(args.workload)
    G, S, n = w.group_size, w.n_stages, w.numel
    cols = w.tensors[0].cols
    rows = n // cols
    print(f"bench: materializing {w.name}: {n} weights", file=sys.stderr, flush=True)
    W = wl.materialize(w).view(rows, cols)
    codes = torch.empty((S, n // 16), dtype=torch.int32, device="cuda")
    scales = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
    zeros = torch.empty((S, n // G), dtype=torch.float32, device="cuda")
    outs = {k: torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda") for k in w.recon_k}
    stream = torch.cuda.current_stream()

    # Calls of one step: (W, rows, cols, codes, scales, zeros, {k: out}) per call.
    if args.per_tensor:
        calls = []
        cflat, sflat, zflat = codes.view(-1), scales.view(-1), zeros.view(-1)
        Wf = W.view(-1)
        for t in w.tensors:
            c = cflat[S * t.offset // 16:S * (t.offset + t.numel) // 16].view(S, t.numel // 16)
            sc = sflat[S * t.offset // G:S * (t.offset + t.numel) // G].view(S, t.numel // G)
            zz = zflat[S * t.offset // G:S * (t.offset + t.numel) // G].view(S, t.numel // G)
            o = {k: outs[k].view(-1)[t.offset:t.offset + t.numel] for k in w.recon_k}
            calls.append((Wf[t.offset:t.offset + t.numel], t.rows, t.cols, c, sc, zz, o))
    else:
        calls = [(W, rows, cols, codes, scales, zeros, outs)]

    step_bytes = construct_bytes(n, G, S) + sum(reconstruct_bytes(n, G, k, 2) for k in w.recon_k)
    flush = (args.flush_mall == "on" or (args.flush_mall == "auto" and step_bytes < 4e9))
    flush_buf = torch.empty(512 << 18, dtype=torch.float32, device="cuda") if flush else None

    def step(evs=None):
        if flush_buf is not None:
            flush_buf.fill_(1.0)
        if evs is not None:
            evs[0].record(stream)
        for Wc, r_, c_, cc, sc, zz, _ in calls:
            rrq.rrq_construct(Wc, r_, c_, G, S, cc, sc, zz, stream)
        if evs is not None:
            evs[1].record(stream)
        for i, k in enumerate(w.recon_k):
            for _, r_, c_, cc, sc, zz, o in calls:
                rrq.rrq_reconstruct(cc, sc, zz, r_, c_, G, S, k, o[k], rrq.RRQ_BF16, stream)
            if evs is not None:
                evs[2 + i].record(stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    print(f"bench: warmup done ({args.warmup} steps)", file=sys.stderr, flush=True)

    events = [[torch.cuda.Event(enable_timing=True) for _ in range(2 + len(w.recon_k))]
              for _ in range(args.steps)]
    torch.cuda.synchronize()
    gc.collect()
    gc.disable()   # no collection pause inside the timed steps
    t0 = time.perf_counter()
    for s in range(args.steps):
        step(events[s])
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    gc.enable()

    cons_ms = [e[0].elapsed_time(e[1]) for e in events]
    rec_ms = {k: [e[1 + i].elapsed_time(e[2 + i]) for e in events] for i, k in enumerate(w.recon_k)}
    mean = lambda xs: sum(xs) / len(xs)
    median = lambda xs: sorted(xs)[len(xs) // 2] if len(xs) % 2 else \
        0.5 * (sorted(xs)[len(xs) // 2 - 1] + sorted(xs)[len(xs) // 2])
    c_ms = mean(cons_ms)
    bf16_gbs = 2 * n / (c_ms * 1e-3) / 1e9
    c_bytes = construct_bytes(n, G, S)
    c_achieved = c_bytes / (c_ms * 1e-3) / 1e9
    recon = {}
    for k in w.recon_k:
        r_ms = mean(rec_ms[k])
        recon[str(k)] = {
            "ms": round(r_ms, 4),
            "ms_median": round(median(rec_ms[k]), 4),
            "ms_min": round(min(rec_ms[k]), 4),
            "gbs_bf16_weights": round(2 * n / (r_ms * 1e-3) / 1e9, 2),
            "hbm_gbs": round(reconstruct_bytes(n, G, k, 2) / (r_ms * 1e-3) / 1e9, 2),
        }
    print(f"bench: construct {c_ms:.3f} ms, {bf16_gbs:.1f} GB/s bf16, {c_achieved:.1f} GB/s HBM",
          file=sys.stderr, flush=True)

    result = {
        "metric": METRIC,
        "value": round(bf16_gbs, 2),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(wall * 1e3 / args.steps, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": w.name,
            "weights": n,
            "tensors": len(w.tensors),
            "group_size": G,
            "n_stages": S,
            "input": "bf16",
            "recon_k": list(w.recon_k),
            "recon_out": "bf16",
            "calls": (f"one call per tensor ({len(calls)} per kernel)" if args.per_tensor
                      else "one flat call per kernel over the whole stack"),
            "mall_flush": flush,
        },
        "construct_ms": round(c_ms, 4),
        "construct_ms_median": round(median(cons_ms), 4),
        "construct_ms_min": round(min(cons_ms), 4),
        "construct_hbm_frac": round(c_achieved / HBM_PEAK_GBS, 4),
        "reconstruct": recon,
        "roofline": {
            "kernel": "construct_kernel<128>",
            "bound": "hbm",
            "achieved": round(c_achieved, 1),
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": round(c_achieved / HBM_PEAK_GBS, 4),
            "traffic": None,
            "bytes_per_launch": c_bytes,
        },
    }
    # Measured HBM traffic of the construct kernel from the committed
    # FETCH_SIZE / WRITE_SIZE profile, only while the kernel source is the one
    # that was profiled.
    from paper_2608_04048_amd import profiling
    rec = profiling.read_traffic_profile(TRAFFIC_PROFILE)
    if (rec is not None and w.name == "qwen3_8b_stack36" and not args.per_tensor
            and rec[0] == profiling.kernel_source_sha256()):
        result["roofline"]["traffic"] = rec[1]
    if not args.per_tensor and len(w.tensors) > 1:
        print("bench: timing one construct call per tensor", file=sys.stderr, flush=True)
        result["per_tensor"] = time_per_tensor(w, W.view(-1), codes, scales, zeros, stream)
    if S >= 2 and not args.no_from_base:
        fb_ms, fb_min = time_from_base(calls, G, S, stream, flush_buf)
        fb_bytes = from_base_bytes(n, G, S)
        result["from_base"] = {
            "kernel": f"construct_kernel<{G}, from base>",
            "ms": round(fb_ms, 4), "ms_min": round(fb_min, 4),
            "gbs_bf16_weights": round(2 * n / (fb_ms * 1e-3) / 1e9, 2),
            "hbm_gbs": round(fb_bytes / (fb_ms * 1e-3) / 1e9, 1),
            "hbm_frac": round(fb_bytes / (fb_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
            "bytes_per_launch": fb_bytes,
            "base": "stage 0 of the package built in the steps",
        }
    if not args.no_pmr:
        print("bench: timing the peak-to-mean side output", file=sys.stderr, flush=True)
        result["pmr"] = time_pmr(w, W, G, S, stream)
    if not args.no_formats:
        print("bench: timing construct in other stage formats", file=sys.stderr, flush=True)
        result["formats"] = time_formats(W, n, G, S, stream)
    if not args.no_linear:
        print("bench: timing rrq_linear decode passes", file=sys.stderr, flush=True)
        result["linear"] = time_linear(w, W.view(-1), codes, scales, zeros, stream)
        print("bench: timing rrq_linear at prefill size", file=sys.stderr, flush=True)
        result["prefill"] = time_prefill()
    if not args.no_stream_probe:
        result["stream_probe"] = stream_probe(min(2 * n, 16 << 30), flush_buf)
        result["construct_frac_of_probe"] = round(c_achieved / result["stream_probe"]["gbs"], 4)
        if not args.per_tensor:
            print("bench: construct-pattern probe", file=sys.stderr, flush=True)
            cp = construct_probe(W, n, G, S, codes, scales, zeros, stream, flush_buf)
            result["stream_probe"]["construct_pattern"] = cp
            result["construct_frac_of_construct_pattern"] = round(c_achieved / cp["gbs"], 4)
            print("bench: reconstruct-pattern probe", file=sys.stderr, flush=True)
            rp = reconstruct_probe(n, G, w.recon_k, codes, scales, zeros, outs, stream, flush_buf)
            result["stream_probe"]["reconstruct_pattern"] = rp
            result["reconstruct_frac_of_reconstruct_pattern"] = {
                str(k): round(rp[str(k)]["ms"] / recon[str(k)]["ms"], 4) for k in w.recon_k}
    if not args.no_cpu_baseline:
        print("bench: timing the CPU oracle", file=sys.stderr, flush=True)
        result["cpu_baseline"] = cpu_baseline(w, W.view(-1), args.cpu_budget, args.cpu_threads)
    print(json.dumps(result), flush=True)
    # Release the device buffers and let queued work drain before the
    # interpreter exits, so that the process ends right after its line.
    del W, codes, scales, zeros, outs, calls, flush_buf
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


if __name__ == "__main__":
    main()
