#!/usr/bin/env python3
"""Benchmark of the BitLinear W1.58A8 hot path (BitNet b1.58, arXiv 2402.17764, Section 2) on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload 70b_decode|7b_decode|3b_decode]

A "step" is one pass of the per-token hot path over one batch of synthetic activations: for every
layer of the workload and every projection shape, per-token int8 activation quantization, the
ternary product and the rescale (M = 1 token for the decode workloads) -- one bitnet_linear_fused
launch per product, or bitnet_quantize_acts + bitnet_linear with --unfused.  The step is captured
once into a HIP graph and replayed, the way a decode loop would run it.  Weight quantization +
packing (Eq. 1-3) happens once per layer before the timed region, as it does for inference, and is
timed separately.  The default workload is the 70B-class feed-forward stack with all 80 layers' packed
weights resident (14.1 GB); the other configurations are extra legs of the same JSON line: the 3B decode
step and decoder chain, the 70B feed-forward chain, batched decode on the 7B shapes, the 13B prefill
GEMM at 2048 and 512 tokens, the 700M-class single layer, the 70B prefill product, and the 5-trit
format against the 2-bit one.  Every input is seeded and synthetic (see paper_2402_17764_amd/synth.py
for the recipe); big tensors are drawn on the device with the same distributions.

Prints ONE JSON line; exits non-zero (after printing it) if any leg failed.
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published
INT8_MFMA_PEAK_TOPS = 5000.0   # MI355X dense int8 MFMA, published (5.0 POP/s)

WORKLOADS = {
    # name: (config index in synth.CONFIGS, M, layers)
    "3b_decode": (1, 1, 26),
    "7b_decode": (2, 1, 32),
    "70b_decode": (4, 1, 80),
}
DEFAULT_WORKLOAD = "70b_decode"

# token counts of the extra legs (the launch inventory below and the legs themselves read these)
BATCHED_DECODE_MS = (1, 8, 16, 32, 64)
BATCHED_DECODE_MS_WS = (128, 256)
BATCHED_DECODE_FUSED_MS = (8,)
GEMM_MS = (2048, 512)
SMALL_LAYER_MS = (1, 16)
PREFILL_70B_M = 4096
LEGS = ["decode_3b_m1", "decoder_chain_3b_m1", "ffn_chain_70b_m1", "batched_decode_7b", "gemm_13b", "layer_700m",
        "prefill_70b_m4096", "trit5_vs_2bit_m1"]

# what the paper itself reports for this path: whole-model figures on other hardware, context only
PAPER_REPORTED = {
    "note": "whole-model numbers from the paper (FasterTransformer + a third-party 2-bit kernel; the GPU of Table 1 / "
            "Figure 2 is not stated, Table 3 is 2x A100 80GB with pipeline parallelism); no per-layer GEMV or GEMM "
            "figure is published, so vs_baseline is null",
    "decode_latency_ms_per_token_fp16_vs_b158 (Table 1)": {"700M": [1.18, 0.96], "1.3B": [1.62, 0.97], "3B": [5.07, 1.87],
                                                            "3.9B": [None, 2.11]},
    "decode_speedup_70b (Figure 2, text)": 4.1,
    "throughput_70b_tokens_per_s_fp16_vs_b158 (Table 3, 2x A100 80GB, seq 512)": [333, 2977],
    "max_batch_70b_fp16_vs_b158 (Table 3)": [16, 176],
    "memory_GB_fp16_vs_b158 (Table 1)": {"700M": [2.08, 0.80], "1.3B": [3.34, 1.14], "3B": [7.89, 2.22], "3.9B": [None, 2.38]},
}


def launch_inventory():
    """Every product launch a default run times, as (leg, entry point, x dtype, M, N, K) with the names of
    paper_2402_17764_amd.binding.ENTRY_* -- N and K as that entry point takes them.  tests/test_dispatch_cpu.py maps
    each to the kernel instantiation it gets and checks that a GPU parity test reaches the same instantiation."""
    from paper_2402_17764_amd import synth
    inv = []
    for wl, leg in ((DEFAULT_WORKLOAD, "headline"), ("3b_decode", "decode_3b_m1")):
        cfg_idx, M, _ = WORKLOADS[wl]
        for (_, K, N) in synth.CONFIGS[cfg_idx]["shapes"]:
            inv.append((leg, "LINEAR_FUSED", "bf16", M, N, K))
    sh = {n: (K, N) for (n, K, N) in synth.CONFIGS[1]["shapes"]}
    H, F = sh["qkv"][0], sh["down"][0]
    inv += [("decoder_chain_3b_m1", "RMSNORM_LINEAR_FUSED", "bf16", 1, sh["qkv"][1], H),
            ("decoder_chain_3b_m1", "LINEAR_FUSED", "bf16", 1, H, H),
            ("decoder_chain_3b_m1", "FFN_GATE_UP_NORM", "bf16", 1, F, H),
            ("decoder_chain_3b_m1", "LINEAR_FUSED", "bf16", 1, H, F)]
    for (_, K, N) in synth.CONFIGS[1]["shapes"]:
        inv.append(("decoder_chain_3b_m1", "LINEAR", "int8", 1, N, K))
    sh = {n: (K, N) for (n, K, N) in synth.CONFIGS[4]["shapes"]}
    H, F = sh["gate_up"][0], sh["down"][0]
    inv += [("ffn_chain_70b_m1", "FFN_GATE_UP_NORM", "bf16", 1, F, H), ("ffn_chain_70b_m1", "LINEAR_FUSED", "bf16", 1, H, F)]
    for (_, K, N) in synth.CONFIGS[2]["shapes"]:
        for M in BATCHED_DECODE_MS + BATCHED_DECODE_MS_WS:
            inv.append(("batched_decode_7b", "LINEAR", "int8", M, N, K))
        for M in BATCHED_DECODE_FUSED_MS:
            if 32 * 16 + M * ((K + 255) // 256) * 256 <= 65536:       # header + int8 rows within the fused kernel's LDS budget
                inv.append(("batched_decode_7b", "LINEAR_FUSED", "bf16", M, N, K))
    for (_, K, N) in synth.CONFIGS[3]["shapes"]:
        for M in GEMM_MS:
            inv.append(("gemm_13b", "LINEAR", "int8", M, N, K))
    for (_, K, N) in synth.CONFIGS[0]["shapes"]:
        for M in SMALL_LAYER_MS:
            inv.append(("layer_700m", "LINEAR", "int8", M, N, K))
            inv.append(("layer_700m", "LINEAR_FUSED", "f32", M, N, K))
    for (_, K, N) in synth.CONFIGS[4]["shapes"]:
        inv.append(("prefill_70b_m4096", "LINEAR", "int8", PREFILL_70B_M, N, K))
    for (K, N) in ((3200, 17280), (8192, 57344)):
        inv.append(("trit5_vs_2bit_m1", "LINEAR", "int8", 1, N, K))
    return inv


def progress(msg):
    """a line on stderr per finished stage, so that a long run (under a profiler, say) is seen to move"""
    print("[bench] " + msg, file=sys.stderr, flush=True)


def fused_supported(B, M, N, K):
    """whether bitnet_linear_fused takes this shape (host-side query, nothing is launched)"""
    try:
        B.entry_describe(B.ENTRY_LINEAR_FUSED, M, N, K, x_dtype=B.BF16)
        return True
    except B.BitnetError:
        return False


def gemv_bytes(M, N, K, out_bytes=2):
    """Algorithmic bytes of one product call: packed 2-bit weights + int8 x + scales + y."""
    return N * K // 4 + M * K + 4 * M + M * N * out_bytes


def measured_traffic(N, K, fused=True):
    """HBM bytes per launch of the M = 1 product on an N x K layer, from the committed rocprofv3 --pmc summary
    (profiles/hbm_traffic.json: FETCH_SIZE + WRITE_SIZE, each scaled by what the counter reads for a plain
    256 MiB copy).  `fused`: the launch that quantizes x itself (linear_decode_2bit without a norm or a gate) or the one on int8
    input (linear_gemv16_2bit, fifth template parameter 0 or 1).  None if the summary has no entry for this launch shape."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        table = json.load(f)
    for key, v in table.get("kernels", {}).items():
        name = "linear_decode_2bit" if fused else "linear_gemv16_2bit"
        if key.startswith(name + "<") and v.get("N") == N and v.get("K") == K:
            params = [p.strip() for p in key[key.index("<") + 1:key.index(">")].split(",")]
            if params[7:9] == ["false", "false"] if fused else len(params) >= 6 and params[5] == "false" and params[4] in ("0", "1"):
                return int(v["fetch_bytes"] + v["write_bytes"])
    return None


def plain_read_floor(torch, buffers, nbytes, stream, args):
    """A kernel that only reads `nbytes` of each buffer (paper_2402_17764_amd/csrc/floors.hip, a library of its own),
    timed like the product: one HIP graph of back-to-back launches over the distinct buffers, best of five launch shapes.
    What the memory system gives a launch of this size when nothing else is done; None if that library is not built."""
    try:
        from paper_2402_17764_amd import floors
        lib = floors.load()
    except Exception:                                     # measurement aid only: the benchmark line does not depend on it
        return None
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    best = None
    for (blocks, loads) in ((256, 4), (256, 8), (512, 2), (512, 4), (1024, 2)):
        def run():
            s = torch.cuda.current_stream().cuda_stream
            for b in buffers:
                lib.read_only_launch(b.data_ptr(), nbytes, sink.data_ptr(), blocks, loads, s)

        ms, _, graph = time_graph(torch, run, max(2, args.warmup // 3), max(5, args.steps // 3), stream)
        del graph
        us = ms * 1e3 / len(buffers)
        if best is None or us < best["us_per_launch"]:
            best = {"us_per_launch": round(us, 3), "GB/s": round(nbytes / (us * 1e-6) / 1e9, 1),
                    "frac_hbm_peak": round(nbytes / (us * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
                    "launch": "%d workgroups x 512 threads, %d loads of 16 bytes in flight per thread" % (blocks, loads)}
    return best


def mfma_only_floor(torch, xq, codes):
    """A loop of v_mfma_i32_32x32x32_i8 from registers and nothing else (csrc/floors.hip: eight accumulator fragments per
    wave, two workgroups of four waves per CU, as the prefill kernel's 128 x 256 tile), on operand registers filled from the
    leg's own x_q and decoded weights (64 x code), and on all-zero operands: what the matrix pipe sustains on data like the
    workload's -- the clock under MFMA load follows the operands' switching activity.  None if the library is not built."""
    try:
        from paper_2402_17764_amd import floors
        lib = floors.load()
    except Exception:
        return None
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    w64 = (codes.reshape(-1)[: 1 << 24] * 64).contiguous()
    xa = xq.reshape(-1)[: 1 << 24].contiguous()
    zeros = torch.zeros(1 << 20, dtype=torch.int8, device="cuda")
    blocks, iters = 512, 20000
    ops = blocks * 4.0 * iters * 8 * 65536
    out = {}
    for tag, a, b in (("workload_operands", xa, w64), ("zero_operands", zeros, zeros)):
        nbytes = min(a.numel(), b.numel())
        s = torch.cuda.current_stream().cuda_stream
        best = None
        for rep in range(3):
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            lib.mfma_only_launch(a.data_ptr(), b.data_ptr(), nbytes, blocks, iters, sink.data_ptr(), s)
            e1.record()
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1)
            best = ms if best is None or ms < best else best
        out[tag + "_TOPS"] = round(ops / (best * 1e-3) / 1e12, 1)
    return out


def make_acts(torch, M, K, gen, seed_channels):
    import numpy as np
    from paper_2402_17764_amd import synth
    x = torch.randn((M, K), device="cuda", generator=gen, dtype=torch.float32)
    ch = torch.from_numpy(synth.outlier_channels(K, config=seed_channels)).cuda()
    x[:, ch] *= synth.OUTLIER_SCALE
    return x.to(torch.bfloat16)


def time_graph(torch, fn, warmup, steps, stream):
    """Capture fn() (launches on the current stream) into a HIP graph; time `steps` replays."""
    with torch.cuda.stream(stream):
        fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        fn()
    # warm-up: at least `warmup` replays and at least 30 ms of them (clocks and caches settle over the first
    # tens of milliseconds of a new kind of load)
    t_w = time.perf_counter()
    done = 0
    while done < max(1, warmup) or time.perf_counter() - t_w < 0.030:
        graph.replay()
        done += 1
        if done % 8 == 0:
            torch.cuda.synchronize()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record()
    for _ in range(steps):
        graph.replay()
    e1.record()
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3
    return e0.elapsed_time(e1) / steps, wall_ms / steps, graph


def _time_cpu(fn, seconds_target):
    fn()
    t0 = time.perf_counter()
    fn()
    per = time.perf_counter() - t0
    reps = max(1, min(200, int(seconds_target / max(per, 1e-6))))
    t0 = time.perf_counter()
    for _ in range(reps):
        fn()
    return (time.perf_counter() - t0) / reps, reps


def cpu_baseline(cfg_idx, M, seconds_target=8.0):
    """The oracle as it stands, timed on the host cores on a bounded sample of the headline workload: the per-token
    path (activation quantization, integer product, rescale) over one layer set whose matrices keep every eighth of
    their rows when they exceed 150 M weights (the work per byte of a weight-streaming product does not depend on the
    row count); same algorithmic-bytes unit as the GPU value.  `other_configs` holds the same measurement for the
    remaining benchmark configurations, each on a stated sample, and the oracle's weight quantization."""
    import numpy as np
    import oracle
    from paper_2402_17764_amd import synth

    def layer_set(ci, M, max_weights=150e6, tokens=None):
        cfg = synth.CONFIGS[ci]
        layers, nbytes, ops = [], 0, 0
        for t, (name, K, N) in enumerate(cfg["shapes"]):
            while N * K > max_weights:
                N = N // 8
            W = synth.weights(N, K, config=ci, layer=0, tensor=t)
            codes, gamma = oracle.quantize_weights(W)
            x, _ = synth.activations(tokens or M, K, config=ci, layer=0, tensor=100 + t, bf16=True)
            layers.append((x, codes, gamma, N, K))
            nbytes += gemv_bytes(tokens or M, N, K)
            ops += 2 * (tokens or M) * N * K
            del W

        def one_pass():
            for (x, codes, gamma, N, K) in layers:
                xq, sx = oracle.quantize_acts(x)
                acc = oracle.ternary_matmul(xq, codes)
                oracle.rescale(acc, gamma, sx)
        return one_pass, nbytes, ops, [(N, K) for (_, _, _, N, K) in layers]

    cfg = synth.CONFIGS[cfg_idx]
    one_pass, nbytes, _, dims = layer_set(cfg_idx, M)
    dt, reps = _time_cpu(one_pass, seconds_target)
    out = {
        "value": round(nbytes / dt / 1e9, 3), "unit": "GB/s", "cores": oracle.num_threads(), "kind": "oracle",
        "sample": "one layer set of %s at M=%d with the row counts cut to %s (N x K; %.0f MB of algorithmic bytes per pass), "
                  "activation quantization + integer product + rescale, mean of %d passes; sampled, not extrapolated"
                  % (cfg["name"], M, dims, nbytes / 1e6, reps),
    }
    other = {}
    for (tag, ci, m, tok, cap) in (("700m_layer_m1", 0, 1, None, 150e6), ("700m_layer_m16", 0, 16, None, 150e6),
                                   ("3b_decode_m1", 1, 1, None, 150e6), ("7b_decode_m1", 2, 1, None, 150e6),
                                   ("7b_decode_m64", 2, 64, None, 12e6), ("13b_prefill_m512", 3, 512, 16, 12e6)):
        if ci == cfg_idx and m == M:
            continue
        fn, nb, ops, dims = layer_set(ci, m, max_weights=cap, tokens=tok)
        dt, reps = _time_cpu(fn, 1.5)
        other[tag] = {"GB/s": round(nb / dt / 1e9, 3), "TOPS": round(ops / dt / 1e12, 5), "passes": reps,
                      "sample": "one layer set, rows cut to %s%s" % (dims, ", %d of %d tokens" % (tok, m) if tok else "")}
    W = synth.weights(4096, 4096, config=2, layer=0, tensor=1)
    dt, reps = _time_cpu(lambda: oracle.quantize_weights(W), 1.5)
    other["weight_quant_4096x4096"] = {"GB/s": round(8.25 * W.size / dt / 1e9, 3), "passes": reps,
                                       "note": "Eq. (1)-(3) without packing, 8.25 algorithmic bytes per weight"}
    out["other_configs"] = other
    return out


def quant_bytes(N, K):
    """HBM bytes per fp32 weight of quantizing and packing an N x K matrix: the reads of W and the packed write."""
    return 4.25 if N * K * 4 >= 96 << 20 else 8.25


def decode_workload(torch, B, synth, gen, stream, args, workload):
    """One decode workload: weights drawn, quantized and packed through the library (timed per call), the step
    (every product of every layer, M tokens) as one HIP graph, and the same for the dominant product alone."""
    cfg_idx, M, L = WORKLOADS[workload]
    cfg = synth.CONFIGS[cfg_idx]
    shapes = cfg["shapes"]
    packed, wq_ms, wq_bytes = {}, 0.0, 0
    ws_bytes = max(B.quantize_weights_workspace(N, K) for (_, K, N) in shapes)
    workspace = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    for l in range(L):
        for (name, K, N) in shapes:
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            if l == 0:
                B.quantize_weights(W, workspace=workspace)          # warm the code path
                torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            packed[(l, name)] = B.quantize_weights(W, workspace=workspace)
            e1.record()
            torch.cuda.synchronize()
            wq_ms += e0.elapsed_time(e1)
            wq_bytes += int(N * K * quant_bytes(N, K))
            del W
    progress("%s: %d tensors quantized and packed" % (workload, L * len(shapes)))
    acts = {K: make_acts(torch, M, K, gen, cfg_idx) for K in sorted({K for (_, K, _) in shapes})}
    xq = {K: torch.empty((M, K), dtype=torch.int8, device="cuda") for K in acts}
    sx = {K: torch.empty(M, dtype=torch.float32, device="cuda") for K in acts}
    ys = {name: torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for (name, K, N) in shapes}

    def step():
        for l in range(L):
            for (name, K, N) in shapes:
                p, g = packed[(l, name)]
                if args.unfused:
                    B.quantize_acts(acts[K], xq=xq[K], sx=sx[K])
                    B.linear(xq[K], sx[K], p, g, N, y_dtype=B.BF16, y=ys[name])
                else:
                    B.linear_fused(acts[K], p, g, N, y_dtype=B.BF16, y=ys[name])

    ms_per_step, _, _ = time_graph(torch, step, args.warmup, args.steps, stream)
    step_bytes = L * sum(gemv_bytes(M, N, K) for (_, K, N) in shapes)
    value = step_bytes / (ms_per_step * 1e-3) / 1e9
    progress("%s: step timed, %.4f ms" % (workload, ms_per_step))

    # per-shape launch time (each shape alone, one launch per layer on that layer's own weights) and the roofline of
    # the dominant kernel: the product on the shape that moves the most bytes
    per_shape = {}
    for (name, K, N) in shapes:
        B.quantize_acts(acts[K], xq=xq[K], sx=sx[K])

        def only(name=name, K=K, N=N):
            for l in range(L):
                p, g = packed[(l, name)]
                if args.unfused:
                    B.linear(xq[K], sx[K], p, g, N, y_dtype=B.BF16, y=ys[name])
                else:
                    B.linear_fused(acts[K], p, g, N, y_dtype=B.BF16, y=ys[name])

        ms, _, _ = time_graph(torch, only, args.warmup, args.steps, stream)
        us = ms * 1e3 / L
        nb = gemv_bytes(M, N, K)
        per_shape[name] = {"K": K, "N": N, "us_per_launch": round(us, 3), "bytes_per_launch": nb,
                           "GB/s": round(nb / (us * 1e-6) / 1e9, 1), "frac_hbm_peak": round(nb / (us * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
                           "traffic": measured_traffic(N, K, fused=not args.unfused)}
    dname, dK, dN = max(shapes, key=lambda s: s[1] * s[2])
    d = per_shape[dname]
    for (name, K, N) in shapes:
        floor = plain_read_floor(torch, [packed[(l, name)][0] for l in range(L)], N * K // 4, stream, args)
        per_shape[name]["plain_read"] = floor
        if floor:
            per_shape[name]["frac_of_plain_read_rate"] = round(floor["us_per_launch"] / per_shape[name]["us_per_launch"], 4)
    progress("%s: per-shape launches and the plain-read floor timed" % workload)
    roofline = {
        "bound": "hbm", "kernel": "linear_gemv16_2bit" if args.unfused else "linear_decode_2bit", "shape": "%s K=%d N=%d M=%d" % (dname, dK, dN, M),
        "achieved": d["GB/s"], "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": d["frac_hbm_peak"],
        "bytes_per_launch": d["bytes_per_launch"], "us_per_launch": d["us_per_launch"], "traffic": d["traffic"],
        "plain_read_of_the_same_weights": d.get("plain_read"), "frac_of_plain_read_rate": d.get("frac_of_plain_read_rate"),
        "traffic_source": "profiles/hbm_traffic.json: rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this launch, "
                          "committed with the tree (not re-measured in this run)",
    }
    return {
        "value": round(value, 1), "ms_per_step": round(ms_per_step, 5), "bytes_per_step": step_bytes,
        "pct_hbm_peak": round(100.0 * value / HBM_PEAK_GBS, 2), "roofline": roofline, "per_shape": per_shape,
        "workload": "%s: %s, M=%d, %d layer sets x %s, bf16 in/out, 2-bit packed weights, %.2f GB of packed weights resident"
                    % (workload, cfg["name"], M, L, [(n, k, nn) for (n, k, nn) in shapes],
                       L * sum(N * K // 4 for (_, K, N) in shapes) / 1e9),
        "launch": "HIP graph replay of %d x %s" % (L * len(shapes), "(bitnet_quantize_acts + bitnet_linear)"
                                                     if args.unfused else "bitnet_linear_fused"),
        "weight_quant": {"ms_per_pass": round(wq_ms, 3), "tensors": L * len(shapes),
                         "ms_per_tensor_mean": round(wq_ms / (L * len(shapes)), 4),
                         "GB/s": round(wq_bytes / (wq_ms * 1e-3) / 1e9, 1),
                         "note": "quantize + pack of every layer; bytes per weight: 4.25 where the matrix is read once (96 MiB and more), else 8.25"},
    }


def ffn_chain_70b_leg(torch, B, synth, gen, stream, args, layers=80):
    """One token through the feed-forward halves of all 80 layers of the 70B-class model, every layer's packed
    weights resident (14.1 GB), as one HIP graph of two launches per layer: the merged gate/up projection with
    RMSNorm + quantization in front and the SwiGLU gate in its epilogue, then the down projection with absmax
    quantization in front.  The attention half (QKV, attention, O) is not in the workload's shape list and is
    left out; residual additions likewise."""
    shapes = {name: (K, N) for (name, K, N) in synth.CONFIGS[4]["shapes"]}
    H, N_gu = shapes["gate_up"]
    F = shapes["down"][0]
    assert N_gu == 2 * F and shapes["down"][1] == H
    packs = []
    for l in range(layers):
        d = {}
        for name, (K, N) in shapes.items():
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            d[name] = B.quantize_weights(W)
            del W
        packs.append(d)
    x0 = make_acts(torch, 1, H, gen, 4)
    gain = torch.ones(H, dtype=torch.float32, device="cuda")
    h_f = torch.empty((1, F), dtype=torch.bfloat16, device="cuda")
    y_d = [torch.empty((1, H), dtype=torch.bfloat16, device="cuda") for _ in range(2)]

    def run():
        x = x0
        for l, d in enumerate(packs):
            B.ffn_gate_up_fused(x, d["gate_up"][0], d["gate_up"][1], F, norm=True, g=gain, eps=1e-6, h_dtype=B.BF16, h=h_f)
            B.linear_fused(h_f, d["down"][0], d["down"][1], H, y_dtype=B.BF16, y=y_d[l & 1])
            x = y_d[l & 1]

    ms, _, _ = time_graph(torch, run, args.warmup, args.steps, stream)
    nbytes = layers * sum(gemv_bytes(1, N, K) for (K, N) in shapes.values())
    out = {"layers": layers, "launches": 2 * layers, "resident_GB": round(layers * (N_gu * H + H * F) / 4 / 1e9, 2),
           "ms_per_token": round(ms, 4), "us_per_layer": round(ms * 1e3 / layers, 2),
           "GB/s": round(nbytes / (ms * 1e-3) / 1e9, 1), "frac_hbm_peak": round(nbytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
           "note": "ffn_gate_up_fused (RMSNorm in, SwiGLU out) + linear_fused(down) per layer, each layer feeding "
                   "the next; the attention half is not in this workload's shape list"}
    del packs
    torch.cuda.empty_cache()
    return out


def _time_eager(torch, fn, iters, warm_s=0.030, warm_min=3):
    """fn() launched back to back on the current stream, HIP events around `iters` calls; warmed for at least warm_s."""
    t_w = time.perf_counter()
    done = 0
    while done < warm_min or time.perf_counter() - t_w < warm_s:
        fn()
        done += 1
        if done % 8 == 0:
            torch.cuda.synchronize()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(iters):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / iters


def prefill_70b_leg(torch, B, synth, gen, stream, args):
    """The 70B-class FFN shapes at M = 4096 (the prefill end of the last configuration's sweep) and the one-off weight
    quantization + packing time per layer."""
    res = {}
    M = PREFILL_70B_M
    for (name, K, N) in synth.CONFIGS[4]["shapes"]:
        wq_ms, pack = [], None
        for l in range(4):
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            pack = B.quantize_weights(W)
            e1.record()
            torch.cuda.synchronize()
            if l >= 1:
                wq_ms.append(e0.elapsed_time(e1))
            del W
        xp = make_acts(torch, M, K, gen, 4)
        xq, sx = B.quantize_acts(xp)
        yp = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        p0, g0 = pack
        us_p = _time_eager(torch, lambda: B.linear(xq, sx, p0, g0, N, y_dtype=B.BF16, y=yp), 5)
        us_q = time_quantize_acts(torch, B, xp, stream)
        tops = 2.0 * M * N * K / (us_p * 1e-6) / 1e12
        res[name] = {"K": K, "N": N, "M": M, "us_linear": round(us_p, 1), "us_quantize_acts": round(us_q, 1), "TOPS": round(tops, 1),
                     "frac_int8_mfma_peak": round(tops / INT8_MFMA_PEAK_TOPS, 4),
                     "weight_quant_ms_per_layer": round(min(wq_ms), 3),
                     "weight_quant_GB/s": round(quant_bytes(N, K) * N * K / (min(wq_ms) * 1e-3) / 1e9, 1)}
        del pack, xq, sx, yp, xp
        torch.cuda.empty_cache()
    return res


def small_layer_leg(torch, B, synth, gen, stream, args):
    """The 700M-class single layer (1536 -> 4096, fp32 activations) at M = 1 and 16: the one-launch fused entry point
    and the two-call route, each replayed over enough distinct layers to exceed the memory-side cache; plus its weight
    quantization.  A 1.5 MB weight stream is 0.2 us at the HBM peak: these launches are latency-bound."""
    res = {}
    for (name, K, N) in synth.CONFIGS[0]["shapes"]:
        layers = 400                                   # 630 MB of packed weights
        packs, wq = [], []
        for l in range(layers):
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            if l in (5, 6, 7):
                torch.cuda.synchronize()
                e0 = torch.cuda.Event(enable_timing=True)
                e1 = torch.cuda.Event(enable_timing=True)
                e0.record()
                packs.append(B.quantize_weights(W))
                e1.record()
                torch.cuda.synchronize()
                wq.append(e0.elapsed_time(e1))
            else:
                packs.append(B.quantize_weights(W))
            del W
        entry = {"K": K, "N": N, "layers": layers, "weight_quant_us": round(min(wq) * 1e3, 1)}
        for M in SMALL_LAYER_MS:
            x = torch.randn((M, K), device="cuda", generator=gen, dtype=torch.float32)
            ch = torch.from_numpy(synth.outlier_channels(K, config=0)).cuda()
            x[:, ch] *= synth.OUTLIER_SCALE
            xq, sx = B.quantize_acts(x)
            y = torch.empty((M, N), dtype=torch.float32, device="cuda")

            def run_fused():
                for (p, g) in packs:
                    B.linear_fused(x, p, g, N, y_dtype=B.F32, y=y)

            def run_two():
                for (p, g) in packs:
                    B.quantize_acts(x, xq=xq, sx=sx)
                    B.linear(xq, sx, p, g, N, y_dtype=B.F32, y=y)

            def run_linear():
                for (p, g) in packs:
                    B.linear(xq, sx, p, g, N, y_dtype=B.F32, y=y)

            nb = gemv_bytes(M, N, K, out_bytes=4)
            e = {}
            for tag, fn in (("linear_fused", run_fused), ("quantize_acts+linear", run_two), ("linear", run_linear)):
                ms, _, gr = time_graph(torch, fn, max(2, args.warmup // 5), max(5, args.steps // 5), stream)
                us = ms * 1e3 / layers
                e[tag] = {"us_per_layer": round(us, 2), "GB/s": round(nb / (us * 1e-6) / 1e9, 1)}
                del gr
            entry["M=%d" % M] = e
        res[name] = entry
        del packs
        torch.cuda.empty_cache()
    return res


def format_leg(torch, B, synth, gen, stream, args):
    """The 5-trits-per-byte format measured against the 2-bit one, same weights: the M = 1 product (bitnet_linear on
    pre-quantized activations) on the dominant 3B shape and the 70B gate/up shape, and the prefill product at 2048
    tokens on the 13B gate/up shape, where 5-trit weights go through bitnet_linear_ws (repacked to 2 bits in the
    workspace, then the MFMA prefill kernel)."""
    res = {}
    for (tag, K, N) in (("3b_gate_up", 3200, 17280), ("70b_gate_up", 8192, 57344)):
        entry = {"K": K, "N": N}
        x = make_acts(torch, 1, K, gen, 1)
        xq, sx = B.quantize_acts(x)
        y = torch.empty((1, N), dtype=torch.bfloat16, device="cuda")
        for (fname, fmt) in (("2bit", B.PACK_2BIT), ("trit5", B.PACK_TRIT5)):
            per = B.packed_bytes(N, K, fmt)
            layers = max(3, int(math.ceil(600e6 / per)))
            g2 = torch.Generator(device="cuda")
            g2.manual_seed(1234)
            packs = []
            for l in range(layers):
                W = torch.randn((N, K), device="cuda", generator=g2, dtype=torch.float32) * synth.SIGMA_W
                packs.append(B.quantize_weights(W, fmt=fmt))
                del W

            def run():
                for (p, g) in packs:
                    B.linear(xq, sx, p, g, N, fmt=fmt, y_dtype=B.BF16, y=y)

            ms, _, _ = time_graph(torch, run, args.warmup, args.steps, stream)
            us = ms * 1e3 / layers
            entry[fname] = {"packed_bytes": per, "us_per_launch": round(us, 2), "GB/s": round(per / (us * 1e-6) / 1e9, 1)}
            del packs
            torch.cuda.empty_cache()
        entry["time_ratio_trit5_over_2bit"] = round(entry["trit5"]["us_per_launch"] / entry["2bit"]["us_per_launch"], 3)
        res[tag] = entry
    # prefill
    M, K, N = 2048, 5120, 27648
    W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
    p2, g2 = B.quantize_weights(W, fmt=B.PACK_2BIT)
    p5, g5 = B.quantize_weights(W, fmt=B.PACK_TRIT5)
    del W
    xq, sx = B.quantize_acts(make_acts(torch, M, K, gen, 3))
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.linear_workspace(M, N, K, fmt=B.PACK_TRIT5), dtype=torch.uint8, device="cuda")
    scratch2 = torch.empty_like(p2)
    us2 = _time_eager(torch, lambda: B.linear(xq, sx, p2, g2, N, y_dtype=B.BF16, y=y), 10)
    us5 = _time_eager(torch, lambda: B.linear_ws(xq, sx, p5, g5, N, ws, fmt=B.PACK_TRIT5, y_dtype=B.BF16, y=y), 10)
    usr = _time_eager(torch, lambda: B.repack_weights(p5, N, K, B.PACK_TRIT5, B.PACK_2BIT, out=scratch2), 10)
    ops = 2.0 * M * N * K
    res["13b_gate_up_m2048"] = {"K": K, "N": N, "M": M, "2bit": {"packed_bytes": p2.numel(), "us_linear": round(us2, 1), "TOPS": round(ops / us2 * 1e-6, 1)},
                                "trit5": {"packed_bytes": p5.numel(), "us_linear_ws": round(us5, 1), "TOPS": round(ops / us5 * 1e-6, 1),
                                          "us_repack_alone": round(usr, 1), "workspace_bytes": ws.numel()},
                                "time_ratio_trit5_over_2bit": round(us5 / us2, 3)}
    return res


def batched_decode_leg(torch, B, synth, gen, stream, args):
    """The transition between decode and prefill: M = 1 ... 64 tokens (and 128, the first prefill-kernel size) on the
    7B-class shapes, bitnet_linear on pre-quantized activations, each shape replayed over enough distinct layers to exceed the memory-side
    cache.  Both rooflines are reported because M = 64 sits near the ridge between them."""
    res = {}
    for (name, K, N) in synth.CONFIGS[2]["shapes"]:
        per = N * K // 4
        layers = max(3, int(math.ceil(550e6 / per)))
        packs = []
        for l in range(layers):
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            packs.append(B.quantize_weights(W))
            del W
        entry = {"K": K, "N": N, "layers": layers}
        for M in BATCHED_DECODE_MS:
            x = make_acts(torch, M, K, gen, 2)
            xq, sx = B.quantize_acts(x)
            y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")

            def run():
                for (p, g) in packs:
                    B.linear(xq, sx, p, g, N, y_dtype=B.BF16, y=y)

            ms, _, graph = time_graph(torch, run, max(2, args.warmup // 5), max(5, args.steps // 5), stream)
            us = ms * 1e3 / layers
            entry["M=%d" % M] = {"us_per_launch": round(us, 2),
                                 "GB/s": round(gemv_bytes(M, N, K) / (us * 1e-6) / 1e9, 1),
                                 "TOPS": round(2.0 * M * N * K / us * 1e-6, 1)}
            del graph
            if M in BATCHED_DECODE_FUSED_MS and fused_supported(B, M, N, K):
                # the same product with the activation quantization inside the launch (bf16 x; up to 16 tokens whose int8
                # rows fit the workgroup's LDS budget)
                def run_fused():
                    for (p, g) in packs:
                        B.linear_fused(x, p, g, N, y_dtype=B.BF16, y=y)

                ms, _, graph = time_graph(torch, run_fused, max(2, args.warmup // 5), max(5, args.steps // 5), stream)
                entry["M=%d" % M]["us_fused"] = round(ms * 1e3 / layers, 2)
                del graph
        # the serving regime just above 64 tokens: small layers still run the token-tiled decode kernels, the others
        # the prefill kernel, timed without and with a split-K workspace (bitnet_linear_ws)
        for M in BATCHED_DECODE_MS_WS:
            x = make_acts(torch, M, K, gen, 2)
            xq, sx = B.quantize_acts(x)
            y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
            ws = torch.empty(max(16, B.linear_workspace(M, N, K)), dtype=torch.uint8, device="cuda")

            def run_plain():
                for (p, g) in packs:
                    B.linear(xq, sx, p, g, N, y_dtype=B.BF16, y=y)

            def run_ws():
                for (p, g) in packs:
                    B.linear_ws(xq, sx, p, g, N, ws, y_dtype=B.BF16, y=y)

            ms_p, _, g1 = time_graph(torch, run_plain, max(2, args.warmup // 5), max(5, args.steps // 5), stream)
            ms_w, _, g2 = time_graph(torch, run_ws, max(2, args.warmup // 5), max(5, args.steps // 5), stream)
            entry["M=%d" % M] = {"us_per_launch": round(ms_p * 1e3 / layers, 2), "us_with_workspace": round(ms_w * 1e3 / layers, 2),
                                 "TOPS": round(2.0 * M * N * K / (min(ms_p, ms_w) * 1e3 / layers) * 1e-6, 1),
                                 "kernel": B.linear_describe(M, N, K)["kernel"]}
            del g1, g2
        res[name] = entry
        del packs
        torch.cuda.empty_cache()
    return res


def decoder_block_leg(torch, B, synth, gen, stream, args, cfg_idx=1, layers=26):
    """Per-token latency of the BitLinear chain of a decoder stack at M = 1, two ways, each one HIP graph:
    "fused": RMSNorm+quantization fused into the QKV and gate/up launches, the SwiGLU gate into the epilogue of the
    gate/up launch, absmax quantization into the O and down launches -- four launches per layer;
    "handover": int8 activations handed from producer to product -- RMSNorm->int8, QKV, quantize, O, RMSNorm->int8,
    gate/up, SwiGLU->int8, down -- eight launches per layer.
    Attention itself and the residual additions are not part of the path and are left out (the attention output
    buffer is quantized as it would arrive)."""
    cfg = synth.CONFIGS[cfg_idx]
    shapes = {name: (K, N) for (name, K, N) in cfg["shapes"]}
    H = shapes["qkv"][0]
    F = shapes["down"][0]
    packs = []
    for l in range(layers):
        d = {}
        for name, (K, N) in shapes.items():
            W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
            d[name] = B.quantize_weights(W)
            del W
        packs.append(d)
    M = 1
    h = make_acts(torch, M, H, gen, cfg_idx)
    att = make_acts(torch, M, H, gen, cfg_idx)
    gain = torch.ones(H, dtype=torch.float32, device="cuda")
    xq_h = torch.empty((M, H), dtype=torch.int8, device="cuda")
    xq_f = torch.empty((M, F), dtype=torch.int8, device="cuda")
    s1 = torch.empty(M, dtype=torch.float32, device="cuda")
    y_qkv = torch.empty((M, shapes["qkv"][1]), dtype=torch.bfloat16, device="cuda")
    y_o = torch.empty((M, H), dtype=torch.bfloat16, device="cuda")
    y_gu = torch.empty((M, 2 * F), dtype=torch.bfloat16, device="cuda")
    y_d = torch.empty((M, H), dtype=torch.bfloat16, device="cuda")
    h_f = torch.empty((M, F), dtype=torch.bfloat16, device="cuda")

    def run_handover():
        x = h
        for d in packs:
            B.rmsnorm_quantize(x, gain, 1e-6, xq=xq_h, sx=s1)
            B.linear(xq_h, s1, d["qkv"][0], d["qkv"][1], shapes["qkv"][1], y_dtype=B.BF16, y=y_qkv)
            B.quantize_acts(att, xq=xq_h, sx=s1)
            B.linear(xq_h, s1, d["o"][0], d["o"][1], H, y_dtype=B.BF16, y=y_o)
            B.rmsnorm_quantize(y_o, gain, 1e-6, xq=xq_h, sx=s1)
            B.linear(xq_h, s1, d["gate_up"][0], d["gate_up"][1], 2 * F, y_dtype=B.BF16, y=y_gu)
            B.swiglu_quantize(y_gu, hq=xq_f, sh=s1)
            B.linear(xq_f, s1, d["down"][0], d["down"][1], H, y_dtype=B.BF16, y=y_d)
            x = y_d

    def run_fused():
        x = h
        for d in packs:
            B.rmsnorm_linear_fused(x, gain, 1e-6, d["qkv"][0], d["qkv"][1], shapes["qkv"][1], y_dtype=B.BF16, y=y_qkv)
            B.linear_fused(att, d["o"][0], d["o"][1], H, y_dtype=B.BF16, y=y_o)
            B.ffn_gate_up_fused(y_o, d["gate_up"][0], d["gate_up"][1], F, norm=True, g=gain, eps=1e-6, h_dtype=B.BF16, h=h_f)
            B.linear_fused(h_f, d["down"][0], d["down"][1], H, y_dtype=B.BF16, y=y_d)
            x = y_d

    ms_f, _, _ = time_graph(torch, run_fused, args.warmup, args.steps, stream)
    ms_h, _, _ = time_graph(torch, run_handover, args.warmup, args.steps, stream)
    nbytes = layers * sum(gemv_bytes(M, N, K) for (K, N) in shapes.values())
    return {"model": cfg["name"], "layers": layers, "launches": 4 * layers, "ms_per_token": round(ms_f, 4),
            "GB/s": round(nbytes / (ms_f * 1e-3) / 1e9, 1),
            "note": "rmsnorm_linear_fused(qkv), linear_fused(o), ffn_gate_up_fused (RMSNorm in, SwiGLU out), "
                    "linear_fused(down) per layer; attention and residual adds excluded",
            "int8_handover": {"launches": 8 * layers, "ms_per_token": round(ms_h, 4),
                              "note": "rmsnorm_quantize, linear(qkv), quantize_acts, linear(o), rmsnorm_quantize, "
                                      "linear(gate_up), swiglu_quantize, linear(down) per layer"}}


def time_quantize_acts(torch, B, x, stream, target_bytes=600e6):
    """bitnet_quantize_acts on copies of x in rotation (more of them than the memory-side cache holds), one HIP
    graph: microseconds per launch.  Launched one by one from Python a call costs more than these kernels run."""
    M, K = x.shape
    n = max(2, min(64, int(math.ceil(target_bytes / (M * K * (x.element_size() + 1))))))
    xs = [x] + [x.clone() for _ in range(n - 1)]
    xqs = [torch.empty((M, K), dtype=torch.int8, device="cuda") for _ in range(n)]
    sx = torch.empty(M, dtype=torch.float32, device="cuda")

    def run():
        for xi, qi in zip(xs, xqs):
            B.quantize_acts(xi, xq=qi, sx=sx)

    ms, _, graph = time_graph(torch, run, 2, 5, stream)
    del graph
    return ms * 1e3 / n


def gemm_one_m(torch, B, synth, gen, args, M, stream):
    """Prefill: M tokens on the 13B-class shapes, bitnet_quantize_acts + bitnet_linear."""
    res = {"M": M, "shapes": {}}
    tot_ops, tot_us = 0.0, 0.0
    for (name, K, N) in synth.CONFIGS[3]["shapes"]:
        W = torch.randn((N, K), device="cuda", generator=gen, dtype=torch.float32) * synth.SIGMA_W
        p, g = B.quantize_weights(W)
        del W
        x = make_acts(torch, M, K, gen, 3)
        xq, sx = B.quantize_acts(x)
        y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        iters = max(5, args.steps // 2)
        t_w = time.perf_counter()                    # clocks settle over the first tens of milliseconds of MFMA load
        done = 0
        while done < max(3, args.warmup) or time.perf_counter() - t_w < 0.030:
            B.linear(xq, sx, p, g, N, y_dtype=B.BF16, y=y)
            done += 1
            if done % 8 == 0:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(iters):
            B.linear(xq, sx, p, g, N, y_dtype=B.BF16, y=y)
        e1.record()
        torch.cuda.synchronize()
        us = e0.elapsed_time(e1) * 1e3 / iters
        us_q = time_quantize_acts(torch, B, x, stream)
        ops = 2.0 * M * N * K
        res["shapes"][name] = {"K": K, "N": N, "us_linear": round(us, 1), "us_quantize_acts": round(us_q, 1),
                               "kernel": B.linear_describe(M, N, K)["kernel"], "TOPS": round(ops / us * 1e-6, 1), "frac_int8_mfma_peak": round(ops / us * 1e-6 / INT8_MFMA_PEAK_TOPS, 4)}
        tot_ops += ops
        tot_us += us
        if name == "gate_up":
            res["mfma_only_loop"] = mfma_only_floor(torch, xq, B.unpack_weights(p, N, K))
        del p, x, xq, y
        torch.cuda.empty_cache()
    res["TOPS"] = round(tot_ops / tot_us * 1e-6, 1)
    if res.get("mfma_only_loop"):
        res["frac_of_mfma_only_loop"] = round(res["TOPS"] / res["mfma_only_loop"]["workload_operands_TOPS"], 4)
    res["roofline"] = {"bound": "mfma", "kernel": "linear_gemm_2bit", "workload": "13B-class layer set, M=%d" % M, "achieved": round(tot_ops / tot_us * 1e-6, 1),
                       "peak": INT8_MFMA_PEAK_TOPS, "unit": "TOP/s", "frac": round(tot_ops / tot_us * 1e-6 / INT8_MFMA_PEAK_TOPS, 4),
                       "mfma_only_loop": res.get("mfma_only_loop"), "frac_of_mfma_only_loop": res.get("frac_of_mfma_only_loop")}
    return res


def gemm_leg(torch, B, synth, gen, stream, args):
    """Prefill on the 13B-class shapes at 2048 tokens (the size the GEMM metric is quoted on) and at 512."""
    return {"M=%d" % M: gemm_one_m(torch, B, synth, gen, args, M, stream) for M in GEMM_MS}


def run_leg_in_child(leg, args):
    """One extra leg in a child process (this process keeps its GPU context and waits).  A leg that fails comes back
    as {"error": ...}; main() then exits non-zero after printing its line."""
    import subprocess
    cmd = [sys.executable, os.path.abspath(__file__), "--only", leg, "--steps", str(args.steps), "--warmup", str(args.warmup)]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    except subprocess.TimeoutExpired:
        return {"error": "timed out"}
    for line in reversed(r.stdout.strip().splitlines()):
        if line.startswith("{"):
            try:
                return json.loads(line)[leg]
            except (ValueError, KeyError):
                break
    return {"error": "exit code %d: %s" % (r.returncode, r.stderr.strip()[-300:])}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default=DEFAULT_WORKLOAD, choices=sorted(WORKLOADS))
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--unfused", action="store_true",
                    help="two launches per product (bitnet_quantize_acts + bitnet_linear) instead of bitnet_linear_fused")
    ap.add_argument("--pmc-calibration", action="store_true",
                    help="also run a plain 256 MiB device copy (torch copy_) three times, so that a rocprofv3 --pmc "
                         "FETCH_SIZE / WRITE_SIZE run of this command contains a kernel of known traffic to scale by")
    ap.add_argument("--no-extras", action="store_true", help="skip the extra legs")
    ap.add_argument("--inprocess", action="store_true",
                    help="run the extra legs inside this process (one process for a profiler to follow); by default "
                         "each runs in a child process, so that a failure there cannot take the headline line with it")
    ap.add_argument("--only", default=None, choices=LEGS,
                    help="run one of the extra legs alone and print only its result (profiling a single kernel family)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on one GPU only (the hot path is a single-GPU kernel; it would shard along "
              "the output features with no collective on the path); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2402_17764_amd import binding as B
    from paper_2402_17764_amd import synth
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    B.load()

    if args.pmc_calibration:
        src = torch.empty(256 << 20, dtype=torch.uint8, device="cuda").random_(0, 255)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    gen = torch.Generator(device="cuda")
    gen.manual_seed(240217764)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())

    def leg_3b():
        r = decode_workload(torch, B, synth, gen, stream, args, "3b_decode")
        torch.cuda.empty_cache()
        return r

    legs = {"decode_3b_m1": leg_3b,
            "decoder_chain_3b_m1": lambda: decoder_block_leg(torch, B, synth, gen, stream, args),
            "ffn_chain_70b_m1": lambda: ffn_chain_70b_leg(torch, B, synth, gen, stream, args),
            "batched_decode_7b": lambda: batched_decode_leg(torch, B, synth, gen, stream, args),
            "gemm_13b": lambda: gemm_leg(torch, B, synth, gen, stream, args),
            "layer_700m": lambda: small_layer_leg(torch, B, synth, gen, stream, args),
            "prefill_70b_m4096": lambda: prefill_70b_leg(torch, B, synth, gen, stream, args),
            "trit5_vs_2bit_m1": lambda: format_leg(torch, B, synth, gen, stream, args)}
    assert sorted(legs) == sorted(LEGS)

    if args.only:
        progress("leg %s alone" % args.only)
        print(json.dumps({"only": args.only, "steps": args.steps, "warmup": args.warmup, args.only: legs[args.only]()}))
        return

    head = decode_workload(torch, B, synth, gen, stream, args, args.workload)
    cfg_idx, M, L = WORKLOADS[args.workload]
    out = {
        "metric": "BitLinear GEMV GB/s (%HBM peak) @M=1", "value": head["value"], "unit": "GB/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": head["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int8",
        "dtype_note": "int8 activations x 2-bit ternary weights on int8 MFMA, int32 accumulation, fp32 rescale, bf16 in / out",
        "data": "synthetic",
        "config": {"workload": head["workload"], "launch": head["launch"], "bytes_per_step": head["bytes_per_step"]},
        "pct_hbm_peak": head["pct_hbm_peak"],
        "roofline": head["roofline"],
        "per_shape": head["per_shape"],
        "weight_quant": head["weight_quant"],
        "paper_reported": PAPER_REPORTED,
    }
    del head
    torch.cuda.empty_cache()

    failed = []
    if not args.no_extras:
        names = list(LEGS)
        if args.workload == "3b_decode":
            names.remove("decode_3b_m1")
        if args.pmc_calibration:
            # under counter collection the 208-launch decoder chain is left out: one such run ended in a hardware
            # exception inside the profiler's queue that no un-profiled or kernel-trace run of the leg shows
            names.remove("decoder_chain_3b_m1")
        for leg in names:
            out[leg] = legs[leg]() if args.inprocess else run_leg_in_child(leg, args)
            progress("leg %s done" % leg)
            if isinstance(out[leg], dict) and "error" in out[leg]:
                failed.append(leg)
        if "gemm_13b" in out and "M=2048" in out["gemm_13b"]:
            out["roofline_gemm_m2048"] = out["gemm_13b"]["M=2048"].get("roofline")
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg_idx, M)
    if failed:
        out["failed_legs"] = failed
    print(json.dumps(out))
    sys.stdout.flush()
    if failed:
        print("bench.py: legs failed: %s" % ", ".join(failed), file=sys.stderr)
        sys.exit(1)


if __name__ == "__main__":
    main()
