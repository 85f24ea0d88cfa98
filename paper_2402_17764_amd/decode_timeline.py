"""Where the time of a decode launch goes: per-workgroup wall-clock stamps inside the two kernels that serve one token, the fused
launches' (decode_kernel.hpp) and the one on int8 input (linear_gemv.hip).

    python -m paper_2402_17764_amd.decode_timeline [70b|3b] [build]

Builds instrumented copies of both (the kernel source with a stamp written by thread 0 of every workgroup at fixed points:
start, weights requested, sums of squares and absmax reduced, activations staged, K loop done, fold done, output stored) into
libraries of their own under _build/, in the launch shapes that the library's own description names for each layer, replays a
HIP graph of launches over distinct weight buffers, and prints the distribution of each stamp over the workgroups of the last
launch, in nanoseconds after that launch's first workgroup started, next to the time per launch.  The instrumented kernels are
a few percent slower than the product kernels (the stamps are stores, and the last one waits for the output store to be
acknowledged).  `build` stops after the build, which needs no GPU.  For tuning and for the figures quoted in the design notes;
nothing in the product path uses it.
"""
import ctypes
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
BUILD = os.path.join(HERE, "_build", "timeline")
NAMES = ["start", "sums of squares reduced", "absmax reduced", "activations staged", "weights requested", "K loop done (wave 0)", "fold done",
         "output stored"]
ORDER = (0, 4, 1, 2, 3, 5, 6, 7)
# (name, fused entry point, N or F, K)
LAYERS = {"70b": [("70B gate_up, norm and gate", "FFN_GATE_UP_NORM", 28672, 8192), ("70B down", "LINEAR_FUSED", 8192, 28672)],
          "3b": [("3B qkv, norm", "RMSNORM_LINEAR_FUSED", 9600, 3200), ("3B o", "LINEAR_FUSED", 3200, 3200),
                 ("3B gate_up, norm and gate", "FFN_GATE_UP_NORM", 8640, 3200), ("3B down", "LINEAR_FUSED", 3200, 8640)]}
STAMP = ("__device__ unsigned long long g_ts[8 * 8192];\n"
         "#define TS(k_) do { __builtin_amdgcn_sched_barrier(0); if (threadIdx.x == 0 && blockIdx.x < 8192) "
         "{ g_ts[blockIdx.x * 8 + (k_)] = wall_clock64(); } __builtin_amdgcn_sched_barrier(0); } while (0)\n")
ACCESS = '''
extern "C" int timeline_read(void* dst, long long bytes) { return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(bitnet::g_ts), bytes); }
extern "C" int timeline_clear() {
    void* p;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(bitnet::g_ts));
    if (e != hipSuccess) return (int)e;
    return (int)hipMemset(p, 0, sizeof(unsigned long long) * 8 * 8192);
}
'''


def stamped(name, stamps):
    """csrc/<name> with `text` put in front of (before) or behind each anchor, which it holds exactly once."""
    src = open(os.path.join(HERE, "csrc", name)).read()
    for anchor, text, before in [("namespace bitnet {\n", STAMP, False)] + stamps:
        assert src.count(anchor) == 1, "anchor not found once: " + anchor[:60]
        src = src.replace(anchor, text + anchor if before else anchor + text)
    return src


def int8_source():
    return stamped("linear_gemv.hip", [
        ("    extern __shared__ uint4 smem[];\n    constexpr int kThreads = kS * kW * kWave;", "\n    TS(0);", False),
        ("    int i = 0;\n    for (; i + kD < items; i += kD) {", "    TS(3);\n", True),
        ("    for (int d = 0; d < kD; ++d) mac(st[d], i + d);\n\n", "    asm volatile(\"\" :: \"v\"(acc[0].x));\n    TS(5);\n\n", False),
        ("            acc[a] = s;\n        }\n    }\n", "    TS(6);\n", False),
        ("            if (n0 < N) store_row4(y, yt, (int64_t)r * N + n0, n0, N, acc[a], scale);\n        }\n    }\n",
         "    __builtin_amdgcn_s_waitcnt(0);\n    TS(7);\n", False)]) + '''
namespace bitnet {      // this library's launches on floating-point input go through the other source
bool launch_decode_fused(bool, bool, bool, const void*, const float*, float, const void*, const float*, int, int64_t, int64_t, int64_t, void*, OutType,
                         hipStream_t, LaunchPlan*, hipError_t*) { return false; }
}
extern "C" int timeline_linear(const void* xq, const float* sx, const void* packed, const float* gamma, long long N, long long K,
                               void* y, void* stream) {
    return (int)bitnet::launch_linear_gemv16_2bit((const int8_t*)xq, sx, packed, gamma, 0, 1, N, K, y, bitnet::OutType::BF16, (hipStream_t)stream, nullptr);
}
''' + ACCESS


def fused_source(layers):
    from paper_2402_17764_amd import binding as B
    src = stamped("decode_kernel.hpp", [
        ("    constexpr int kRsrc = 0x00020000;                  // raw buffer, 32-bit\n", "    TS(0);\n", False),
        ("    // ---- token -> x_q in LDS\n", "    TS(4);\n", True),
        ("        bool decided = true; ", "        TS(1);\n", True),
        ("    float sx[kT];\n", "    TS(2);\n", True),
        ("    // ---- products: column r", "    TS(3);\n", True),
        ("    // ---- lane (g, r) takes row", "    asm volatile(\"\" :: \"v\"(acc[0].x));\n    TS(5);\n", True),
        ("    const int t = r & 3;\n    if (t >= M) return;\n", "    TS(6);\n", True),
        ("        else static_cast<int32_t*>(y)[at] = sum[a] >> 6;\n    }\n", "    __builtin_amdgcn_s_waitcnt(0);\n    TS(7);\n", False)])
    cases = ""
    for i, (_, entry, N, K) in enumerate(layers):
        d = B.entry_describe(getattr(B, "ENTRY_" + entry), 1, N, K)
        r, s, w, depth, xmode = d["params"]
        vecs = -(-K // (64 * s * w * 8))
        norm, pair = "NORM" in entry, "GATE_UP" in entry
        assert vecs <= 4 and xmode == (4 if norm else 2), (entry, N, K, d)
        cases += "        case %d: return (int)bitnet::launch_decode_vecs<%d, %d, %d, %d, %d, true, %s, %s>(c);\n" % (
            i, r, s, w, depth, vecs, str(norm).lower(), str(pair).lower())
    return src + '''
extern "C" int timeline_fused(int layer, const void* x, const float* gain, const void* packed, const float* gamma, long long N, long long K,
                              void* y, void* stream) {
    const bitnet::DecodeCall c{x, gain, 1e-6f, packed, gamma, 0, 1, N, K, y, bitnet::OutType::BF16, (hipStream_t)stream, nullptr};
    switch (layer) {
%s        default: return -1;
    }
}
''' % cases + ACCESS


def build(which):
    from paper_2402_17764_amd.build import HIPCC, FLAGS
    os.makedirs(BUILD, exist_ok=True)
    libs = []
    for name, text in (("int8", int8_source()), ("fused_" + which, fused_source(LAYERS[which]))):
        path, lib = os.path.join(BUILD, name + ".hip"), os.path.join(BUILD, "libtimeline_%s.so" % name)
        if not (os.path.exists(lib) and os.path.exists(path) and open(path).read() == text):
            with open(path, "w") as f:
                f.write(text)
            r = subprocess.run([HIPCC, *FLAGS, "-shared", path, "-o", lib], capture_output=True, text=True)
            if r.returncode != 0:
                os.remove(path)
                raise RuntimeError(r.stderr)
        libs.append(lib)
    return libs


def run(which="70b"):
    import numpy as np
    import torch
    from paper_2402_17764_amd import binding as B
    int8, fused = (ctypes.CDLL(p) for p in build(which))
    vp, i64 = ctypes.c_void_p, ctypes.c_longlong
    int8.timeline_linear.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp]
    fused.timeline_fused.argtypes = [ctypes.c_int, vp, vp, vp, vp, i64, i64, vp, vp]
    for lib in (int8, fused):
        lib.timeline_read.argtypes = [vp, i64]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    for i, (name, entry, N, K) in enumerate(LAYERS[which]):
        rows = 2 * N if "GATE_UP" in entry else N
        layers = max(8, min(40, int(1.2e9 // (rows * K // 4))))
        packs = []
        for _ in range(layers):
            W = torch.randn((rows, K), device="cuda", generator=g) * 0.02
            packs.append(B.quantize_weights(W))
            del W
        x = torch.randn((1, K), device="cuda", generator=g).to(torch.bfloat16)
        gain = 1.0 + 0.1 * torch.randn(K, device="cuda", generator=g)
        xq, sx = B.quantize_acts(x)
        y = torch.empty((1, rows), dtype=torch.bfloat16, device="cuda")
        for lib in (fused, int8):
            def launches(s):
                for (p, gm) in packs:
                    rc = (lib.timeline_fused(i, x.data_ptr(), gain.data_ptr(), p.data_ptr(), gm.data_ptr(), N, K, y.data_ptr(), s) if lib is fused
                          else lib.timeline_linear(xq.data_ptr(), sx.data_ptr(), p.data_ptr(), gm.data_ptr(), rows, K, y.data_ptr(), s))
                    assert rc == 0, rc
            st = torch.cuda.Stream()
            st.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(st):
                launches(st.cuda_stream)
            torch.cuda.synchronize()
            gr = torch.cuda.CUDAGraph()
            with torch.cuda.graph(gr, stream=st):
                launches(st.cuda_stream)
            for _ in range(3):
                gr.replay()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                gr.replay()
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) * 1e3 / (5 * layers)
            assert lib.timeline_clear() == 0
            gr.replay()
            torch.cuda.synchronize()
            buf = np.zeros(8 * 8192, dtype=np.uint64)
            assert lib.timeline_read(buf.ctypes.data, buf.nbytes) == 0
            t = buf.reshape(8192, 8).astype(np.int64)
            t = t[: int((t[:, 0] != 0).sum())]
            r = (t - t[:, 0].min()) * 10.0                              # the wall clock ticks at 100 MHz
            form = B.entry_describe(getattr(B, "ENTRY_" + entry), 1, N, K) if lib is fused else B.linear_describe(1, rows, K)
            print("%s %d -> %d, one token, %s, form %s: %.2f us per launch (instrumented), %d workgroups; ns after the launch's first workgroup started"
                  % (name, K, rows, "bf16 x quantized in the launch" if lib is fused else "int8 x", form["params"], us, len(t)))
            for k in ORDER:
                if (t[:, k] != 0).all():
                    v = r[:, k]
                    print("   %-24s min %6.0f  p10 %6.0f  median %6.0f  p90 %6.0f  max %6.0f"
                          % (NAMES[k], v.min(), np.percentile(v, 10), np.median(v), np.percentile(v, 90), v.max()))
            sys.stdout.flush()
        del packs
        torch.cuda.empty_cache()


if __name__ == "__main__":
    which = sys.argv[1] if len(sys.argv) > 1 else "70b"
    build(which)
    if "build" not in sys.argv[2:]:
        run(which)
