// The fused decode launches for one to four tokens on gfx950: activation quantization (optionally behind RMSNorm), the
// ternary product and, for a merged gate | up matrix, the SwiGLU gate, in one launch whose every wait is worth its time.
// acc[m][n] = sum_k x_q[m][k] * Wt[n][k] exactly in int32 and y = acc * gamma * s_x[m] / 127 (Sections 1-2 of
// arXiv 2402.17764); the arithmetic, hence every bit, is that of the kernels in linear_gemv.hip, which serve more
// tokens, longer rows and int8 input.
//
// What bounds such a launch on all but the largest layers is neither the weight stream nor the arithmetic but the chain
// token -> norm -> absmax -> x_q -> products -> output inside a workgroup, a few hundred instructions that a wave issues one
// by one.  So:
//   * all weights of a wave (kD steps of kR row blocks) are requested before the token has arrived, behind its loads and in
//     front of its arithmetic.  A step's chunk is read through a buffer descriptor of its own: what the wave does not own --
//     quads past the matrix's last column, steps past the last, row blocks past the last -- lies past the descriptor's end and
//     reads as zero codes, so neither the loads nor the products carry a mask or a clamp, and an address is a few scalar
//     instructions;
//   * the token is held in registers (kV 16-byte vectors a thread), zero past its end by the same means;
//   * all tokens go through each reduction together;
//   * a wave's sums are one integer per lane (16 rows x up to 4 columns), folded and gated and stored by all lanes at once.
// A wave issues an instruction every five clocks or so whatever it is, an address path takes a 1 KiB load every 16 to 45, and about
// 32 KiB are in flight per CU: that is what the order of the prologue and the launch shapes (linear_decode.hip) go by.
// Measured, HIP graphs over buffers beyond the caches: 3B QKV with the norm (9600 x 3200) 3.3 us from its first workgroup's start to
// the median workgroup's last store, of which weights requested 0.4, sums of squares 0.7, absmax 1.2, x_q staged 1.4, products done
// 2.6, folded 3.0; gate/up 5.2, O 2.2, down 2.8 (profiles/decode_m1_workgroup_timeline.txt).  linear_gemv16_2bit in its best form -> this,
// back to back 300 x 512 3.5 -> 2.4 us, 4096 x 4096 3.5 -> 3.0, 9600 x 11008 11.1 -> 7.4, 57344 x 8192 with norm and gate 23.2 ->
// 21.1 (117 MB: 5.6 TB/s); the 3B stack (104 launches) 593 -> 448 us.
#pragma once
#include "gemv_common.hpp"

namespace bitnet {

// LDS, in bytes: the waves' absmax of each token; their exact sums of squares (hi, lo), where those are needed; the x_q rows,
// steps * 256 each.  Each wave's plain sums of squares stand where the rows will, and the waves' partial accumulators behind the
// rows where the allocation leaves room, else in their place.  The allocation is that of linear_gemv16_2bit for the same
// parameters: header + max(rows, kW kS kR KiB with a K split).
constexpr int kMaxWaves = 16, kMaxTokens = 4;
constexpr int kDecodeMax = 0, kDecodeExact = kMaxTokens * kMaxWaves * 4, kDecodeHeader = kDecodeExact + 2 * kMaxWaves * 8;

__host__ __device__ constexpr int decode_lds_bytes(int M, int K, int kR, int kS, int kW) {
    const int rows = M * ((K + 255) / 256 * 256), fold = kS > 1 ? kW * kS * kR * 1024 : 0;
    return kDecodeHeader + (rows > fold ? rows : fold);
}

// kR  row blocks per wave (kPair: 2, row block b of the gate half and of the up half)
// kS  waves that split K: wave ws takes steps ws, ws + kS, ...
// kW  row slots per workgroup; kS * kW waves
// kD  steps of weights in flight per wave
// kV  16-byte vectors of a token per thread
// kT  tokens it has room for: 1, 2 or 4 (M <= kT)
template <int kR, int kS, int kW, int kD, int kV, int kT, bool kBf16, bool kNorm, bool kPair>
__global__ __launch_bounds__(kS * kW * kWave) void linear_decode_2bit(
        // 14 dwords (product_flags says why)
        const void* __restrict__ xin, const uint4* __restrict__ packed, const float* __restrict__ gamma,
        const float* __restrict__ gain /* RMSNorm: per-column gain or null */, void* __restrict__ y, int N32, int K32,
        uint32_t flags /* tokens, output type, gamma stride */, float eps) {
#if defined(__HIP_DEVICE_COMPILE__)      // the buffer-resource builtins exist in the device pass only
    static_assert(!kPair || kR == 2, "a gate row block and an up row block per wave");
    static_assert(kS * kW <= kMaxWaves && (kT == 1 || kT == 2 || kT == kMaxTokens), "reduction scratch");
    constexpr int kWaves = kS * kW, kThreads = kWaves * kWave;
    constexpr int kE = kBf16 ? 8 : 4;                  // elements per 16-byte vector
    constexpr int kRsrc = 0x00020000;                  // raw buffer, 32-bit
    extern __shared__ uint4 smem[];
    char* const lds = reinterpret_cast<char*>(smem);
    float* const maxs = reinterpret_cast<float*>(lds + kDecodeMax);
    char* const xlds = lds + kDecodeHeader;
    double* const sums = reinterpret_cast<double*>(xlds);

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);          // scalar: a wave's steps, row blocks and addresses
    const int r = lane & 15, g = lane >> 4;
    const int ws = wave % kS, ww = wave / kS;
    const uint32_t K = (uint32_t)K32, N = (uint32_t)N32;
    const int M = kT <= 2 ? kT : flags_number(flags);
    const OutType yt = flags_out_type(flags);
    const int steps = (int)((K + 255) >> 8);
    const uint32_t last_bytes = ((K + 63) / 64 - 4 * (steps - 1)) * 256;  // one row block's chunk of the last step
    const int rowbytes = steps * 256;
    static_assert(kT * kWaves * 8 <= (kS > 1 ? kW * kS * kR * 1024 : kT * 256 - (kT == 4 ? 256 : 0)), "the sums fit where the rows will be");

    // the tokens (the whole offset in the vector offset: the range check covers that one)
    const uint32_t xbytes = K * (kBf16 ? 2 : 4);
    v4i row[kT][kV];
#pragma unroll
    for (int t = 0; t < kT; ++t) {
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(xin) + (size_t)t * xbytes), 0, t < M ? (int)xbytes : 0, kRsrc);
#pragma unroll
        for (int v = 0; v < kV; ++v) row[t][v] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xr, (v * kThreads + tid) * 16, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);
    // the gain of its columns
    v4i gv[kV][kBf16 ? 2 : 1];
    if (kNorm) {                                       // (without a branch: the wait for the token counts the loads behind it)
        const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gain), 0, gain ? (int)(K * 4) : 0, kRsrc);
#pragma unroll
        for (int v = 0; v < kV; ++v)
#pragma unroll
            for (int h = 0; h < (kBf16 ? 2 : 1); ++h)
                gv[v][h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(gr, (v * kThreads + tid) * (kE * 4) + 16 * h, 0, 0));
    }
    // A load occupies the CU's address path for 16 clocks, whichever wave it is of: all waves' token loads go first.
    __builtin_amdgcn_sched_barrier(0);
    if (kWaves > 1) __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // the weights
    const uint32_t RBh = kPair ? N / 16 : (N + 15) / 16;                // row blocks (of one half)
    const uint64_t step_bytes = (uint64_t)RBh * (kPair ? 2048 : 1024);
    const uint32_t rb0 = kPair ? blockIdx.x * kW + ww : (blockIdx.x * kW + ww) * kR;
    const char* wbase = reinterpret_cast<const char*>(packed) + step_bytes * (uint32_t)ws;
    int step = ws;                                                      // of the next load
    struct Stage { v4i w[kR]; };
    auto load = [&](Stage& s) {
        const uint32_t bytes = step < steps - 1 ? 1024u : step == steps - 1 ? last_bytes : 0u;
#pragma unroll
        for (int a = 0; a < kR; ++a) {
            const uint32_t rb = kPair ? rb0 + a * RBh : rb0 + a;
            const bool mine = kPair ? rb0 < RBh : rb < RBh;
            const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wbase + (uint64_t)rb * bytes), 0, mine ? (int)bytes : 0, kRsrc);
            s.w[a] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, 0, 2 /* nt: read once */));
        }
        wbase += step_bytes * kS;
        step += kS;
    };
    Stage st[kD];
#pragma unroll
    for (int d = 0; d < kD; ++d) load(st[d]);
    // the output scales, as vector loads: scalar ones would share a counter with the LDS
    float gm[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) {
        const uint32_t rb = kPair ? min(rb0, RBh - 1) + a * RBh : min(rb0 + a, RBh - 1);
        const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gamma + (flags_gstride(flags) ? rb : 0u)), 0, 4, kRsrc);
        gm[a] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(gr, 0, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- token -> x_q in LDS
    auto expand = [&](const v4i& q, float (&f)[kE]) {
        const uint32_t u[4] = {(uint32_t)q.x, (uint32_t)q.y, (uint32_t)q.z, (uint32_t)q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (kBf16) {
                f[2 * e] = __uint_as_float(u[e] << 16);
                f[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
            } else {
                f[e] = __uint_as_float(u[e]);
            }
        }
    };
    float rms[kT];
    if (kNorm) {
        // the sum of squares in plain fp64 (the squares are exact); it decides r except for a token in half a million
        const double inv_K = 1.0 / (double)K;
#pragma unroll
        for (int t = 0; t < kT; ++t) {
            double s[2] = {0.0, 0.0};
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                float f[kE];
                expand(row[t][v], f);
#pragma unroll
                for (int e = 0; e < kE; ++e) s[e & 1] = __builtin_fma((double)f[e], (double)f[e], s[e & 1]);
            }
            const double S = wave_sum_f64(s[0] + s[1]);
            if (lane == 0) sums[t * kMaxWaves + wave] = S;
        }
        __syncthreads();
        bool decided = true;                                            // the same for all threads
#pragma unroll
        for (int t = 0; t < kT; ++t) {
            double S[kWaves];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) S[w] = sums[t * kMaxWaves + w];
#pragma unroll
            for (int n = 1; n < kWaves; n *= 2)
#pragma unroll
                for (int w = 0; w + n < kWaves; w += 2 * n) S[w] += S[w + n];
            const bool here = rms_from_rounded_sum(S[0], inv_K, eps, &rms[t]);
            decided = (here || t >= M) && decided;                      // the sum 0 of a token that is not there is undecided with eps = 0
        }
        if (__builtin_expect(!decided, 0)) {
            // the exact sums, from memory: nothing of this can be worked out ahead of the branch
            double* const hi = reinterpret_cast<double*>(lds + kDecodeExact);
#pragma unroll 1
            for (int t = 0; t < M; ++t) {
                const v4i* x = reinterpret_cast<const v4i*>(static_cast<const char*>(xin) + (size_t)t * xbytes);
                dd acc{0.0, 0.0};
#pragma unroll 1
                for (uint32_t v = tid; v < K / kE; v += kThreads) {
                    float f[kE];
                    expand(x[v], f);
#pragma unroll
                    for (int e = 0; e < kE; ++e) dd_add_double(acc, (double)f[e] * (double)f[e]);
                }
                const dd w = wave_sum_dd(acc);
                if (lane == 0) { hi[wave] = w.hi; hi[kMaxWaves + wave] = w.lo; }
                __syncthreads();
                dd total{hi[0], hi[kMaxWaves]};
#pragma unroll 1
                for (int q = 1; q < kWaves; ++q) dd_add_dd(total, dd{hi[q], hi[kMaxWaves + q]});
                const float exact = (float)(1.0 / sqrt((total.hi + total.lo) / (double)K + (double)eps));
#pragma unroll
                for (int u = 0; u < kT; ++u) rms[u] = u == t ? exact : rms[u];
                __syncthreads();
            }
        }
    }
    // what gets quantized: the element, or (x * r) * gain
    auto values = [&](int t, int v, float (&f)[kE]) {
        expand(row[t][v], f);
        if (kNorm) {
#pragma unroll
            for (int e = 0; e < kE; ++e) f[e] = f[e] * rms[t];
#pragma unroll
            for (int e = 0; e < kE; ++e) f[e] = gain ? f[e] * __int_as_float(gv[v][e / 4][e % 4]) : f[e];
        }
    };
#pragma unroll
    for (int t = 0; t < kT; ++t) {
        float amax = 0.0f;
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            float f[kE];
            values(t, v, f);
#pragma unroll
            for (int e = 0; e < kE; ++e) amax = fmaxf(amax, fabsf(f[e]));
        }
        amax = wave_max_nonneg(amax);
        if (lane == 0) maxs[t * kMaxWaves + wave] = amax;
    }
    __syncthreads();
    float sx[kT];
#pragma unroll
    for (int t = 0; t < kT; ++t) {
        float m[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m[w] = maxs[t * kMaxWaves + w];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) m[0] = fmaxf(m[0], m[w]);
        sx[t] = fmaxf(m[0], kEps);
        const float inv = kQb / sx[t];                                  // one IEEE division per token
        uint32_t* const out = reinterpret_cast<uint32_t*>(xlds + t * rowbytes);
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            if (t >= M || (v * kThreads + tid) * kE >= rowbytes) continue;
            float f[kE];
            values(t, v, f);
#pragma unroll
            for (int h = 0; h < kE / 4; ++h)
                out[(v * kThreads + tid) * (kE / 4) + h] = pack4_quantized(f[4 * h], f[4 * h + 1], f[4 * h + 2], f[4 * h + 3], inv);
        }
    }
    __syncthreads();

    // ---- products: column r of the MFMA is token r % kT, so that every lane ends up with sums of a token
    v4i acc[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) acc[a] = (v4i){0, 0, 0, 0};
    const char* const xl = xlds + min(r % kT, M - 1) * rowbytes + g * 64;
    struct XStage { v4i x[4]; };
    auto read_x = [&](XStage& s, int item) {           // steps past the last meet zero codes
        const char* const p = xl + min(ws + item * kS, steps - 1) * 256;
#pragma unroll
        for (int j = 0; j < 4; ++j) s.x[j] = *reinterpret_cast<const v4i*>(p + j * 16);
    };
    auto mac = [&](const Stage& s, const XStage& x) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int a = 0; a < kR; ++a)
                acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(decode_word_masked((uint32_t)s.w[a][j], 0xC0C0C0C0u), x.x[j], acc[a], 0, 0, 0);
    };
    const int items = ((steps + kS - 1) / kS + kD - 1) / kD * kD;
    XStage xs[2];                                      // one step ahead: an LDS read takes as long as a chunk's products
    read_x(xs[0], 0);
    int i = 0;
    for (; i + kD < items; i += kD) {
#pragma unroll
        for (int d = 0; d < kD; ++d) {
            read_x(xs[(d + 1) & 1], i + d + 1);
            mac(st[d], xs[d & 1]);
            __builtin_amdgcn_sched_barrier(0);         // the refill of a stage right behind its use
            load(st[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (kD & 1) xs[0] = xs[1];
    }
#pragma unroll
    for (int d = 0; d < kD; ++d) {
        if (d + 1 < kD) read_x(xs[(d + 1) & 1], i + d + 1);
        mac(st[d], xs[d & 1]);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- lane (g, r) takes row 4 g + (r >> 2) of the row block, token r & 3 (of which there are M)
    int sum[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) sum[a] = r < 8 ? (r < 4 ? acc[a].x : acc[a].y) : (r < 12 ? acc[a].z : acc[a].w);
    if (kS > 1) {
        const int rows = M * rowbytes, need = (kS - 1) * kW * kR * kWave * 4;
        const bool behind = rows + need <= decode_lds_bytes(M, K32, kR, kS, kW) - kDecodeHeader;
        int* const fold = reinterpret_cast<int*>(xlds + (behind ? rows : 0));
        if (!behind) __syncthreads();                  // every wave is done with the rows
        if (ws > 0) {
#pragma unroll
            for (int a = 0; a < kR; ++a) fold[((ww * (kS - 1) + ws - 1) * kR + a) * kWave + lane] = sum[a];
        }
        __syncthreads();
        if (ws > 0) return;
#pragma unroll
        for (int w = 0; w < kS - 1; ++w)
#pragma unroll
            for (int a = 0; a < kR; ++a) sum[a] += fold[((ww * (kS - 1) + w) * kR + a) * kWave + lane];
    }
    const int t = r & 3;
    if (t >= M) return;
    float s = sx[0];
#pragma unroll
    for (int u = 1; u < kT; ++u) s = t == u ? sx[u] : s;
    float h[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) h[a] = (float)(sum[a] >> 6) * ((gm[a] * s) / kQb);     // the decode factor 64 goes exactly
    if (kPair) h[0] = swiglu_one(h[0], h[kR - 1]);
#pragma unroll
    for (int a = 0; a < (kPair ? 1 : kR); ++a) {
        const uint32_t n = (rb0 + a) * 16 + 4 * g + (r >> 2);
        if (n >= N) continue;
        const size_t at = (size_t)t * N + n;
        if (yt == OutType::BF16) static_cast<uint16_t*>(y)[at] = f32_to_bf16(h[a]);
        else if (yt == OutType::F32) static_cast<float*>(y)[at] = h[a];
        else static_cast<int32_t*>(y)[at] = sum[a] >> 6;
    }
#endif
}

// ---------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------
struct DecodeForm { int r, s, w, d; };                 // kR, kS, kW, kD
struct DecodeCall {
    const void* x; const float* gain; float eps; const void* packed; const float* gamma; int gstride;
    int64_t M, N /* kPair: F */, K; void* y; OutType yt; hipStream_t stream; LaunchPlan* plan;
};
constexpr int kDecodeMaxVecs = 4;                      // 16-byte vectors of a token per thread that forms are built for
constexpr int decode_vecs(int64_t K, int threads, bool bf16) { return (int)((K + threads * (bf16 ? 8 : 4) - 1) / (threads * (bf16 ? 8 : 4))); }

template <int kR, int kS, int kW, int kD, int kV, bool kBf16, bool kNorm, bool kPair>
static hipError_t launch_decode_vecs(const DecodeCall& c) {
    const int rb = (int)ceil_div(c.N, kRowsPerBlock);
    const dim3 grid((unsigned)ceil_div(rb, kPair ? kW : kW * kR)), block(kS * kW * kWave);
    const size_t lds = decode_lds_bytes((int)c.M, (int)c.K, kR, kS, kW);
    if (c.plan) {
        c.plan->set(kPair ? "decode_pair" : "decode", {kR, kS, kW, kD, (kNorm ? 4 : 2) + (kBf16 ? 0 : 1)}, grid.x, 1, block.x, lds, 1);
        return hipSuccess;
    }
    const uint32_t flags = product_flags(c.gstride, c.yt) | (uint32_t)c.M << 4;
    const uint4* p = static_cast<const uint4*>(c.packed);
#define GO(T_) hipLaunchKernelGGL((linear_decode_2bit<kR, kS, kW, kD, kV, T_, kBf16, kNorm, kPair>), grid, block, lds, c.stream, c.x, p, c.gamma, c.gain, c.y, \
                                  (int)c.N, (int)c.K, flags, c.eps)
    if (c.M == 1) GO(1);
    else if (c.M == 2) GO(2);
    else GO(4);
#undef GO
    return hipGetLastError();
}

// one launch shape for layers of kMin ... kMax K steps: a kernel for every number of vectors that such rows have
template <int kR, int kS, int kW, int kD, int kMin, int kMax, bool kBf16, bool kNorm, bool kPair>
static hipError_t launch_decode_shape(const DecodeCall& c) {
    constexpr int kLo = decode_vecs((kMin - 1) * 256 + 16, kS * kW * kWave, kBf16), kHi = decode_vecs(kMax * 256, kS * kW * kWave, kBf16);
    const int v = decode_vecs(c.K, kS * kW * kWave, kBf16);
#define V(V_) if constexpr (kLo <= V_ && V_ <= kHi) { if (v == V_) return launch_decode_vecs<kR, kS, kW, kD, V_, kBf16, kNorm, kPair>(c); }
    V(1) V(2) V(3) V(4)
#undef V
    return hipErrorInvalidDeviceFunction;
}

// The launch shapes, and the K steps of the layers that each is chosen for (linear_decode.hip).
template <bool kBf16, bool kNorm, bool kPair>
hipError_t launch_decode(const DecodeForm& f, const DecodeCall& c) {
#define SHAPE(R_, S_, W_, D_, MIN_, MAX_) \
    if (f.r == R_ && f.s == S_ && f.w == W_ && f.d == D_) return launch_decode_shape<R_, S_, W_, D_, MIN_, MAX_, kBf16, kNorm, kPair>(c)
    if constexpr (kPair) {
        SHAPE(2, 4, 1, 2, 1, 8);
        SHAPE(2, 8, 1, 2, 9, 64);
        SHAPE(2, 4, 2, 2, 5, 64);
        SHAPE(2, 4, 3, 2, 24, 96);                     // twelve waves hold rows of 96 steps, sixteen of 128
        SHAPE(2, 2, 4, 4, 24, 64);
        SHAPE(2, 4, 4, 2, 33, 128);
        SHAPE(2, 1, 4, 4, 1, 23);
        SHAPE(2, 1, 4, 5, 5, 23);
        SHAPE(2, 1, 8, 4, 1, 64);
        SHAPE(2, 1, 8, 5, 5, 64);
    } else {
        SHAPE(1, 4, 1, 2, 1, 8);
        SHAPE(1, 4, 1, 4, 9, 16);
        SHAPE(1, 8, 1, 2, 17, 64);
        SHAPE(1, 8, 1, 3, 17, 64);
        SHAPE(1, 8, 1, 5, 17, 64);
        SHAPE(1, 1, 4, 4, 1, 23);
        SHAPE(1, 1, 4, 5, 5, 23);
        SHAPE(1, 2, 2, 4, 5, 8);
        SHAPE(1, 4, 2, 4, 9, 63);
        SHAPE(1, 4, 2, 5, 9, 63);
        SHAPE(1, 8, 2, 2, 64, 128);
        SHAPE(1, 2, 4, 4, 5, 64);
        SHAPE(1, 1, 8, 4, 1, 64);
        SHAPE(1, 1, 8, 5, 5, 64);
        SHAPE(1, 1, 12, 4, 24, 96);
        SHAPE(2, 1, 8, 2, 1, 3);
        SHAPE(2, 1, 8, 4, 24, 64);
    }
#undef SHAPE
    return hipErrorInvalidDeviceFunction;
}

}  // namespace bitnet
