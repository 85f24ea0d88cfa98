// Per-token absmax quantization of activations to int8 (Section 2 of arXiv 2402.17764: activations
// are scaled per token into [-Q_b, Q_b], Q_b = 127, with no zero point).
//
// One workgroup per token.  The token is read once into registers (16-byte loads), the absmax is
// reduced with DPP steps and scalar reads inside each wave and through LDS across waves, then the same
// registers are scaled, rounded (ties to even) and written as packed int8; rows of any length and alignment
// take the same loads at element alignment.  Tokens too long for the register budget take a two-sweep path that
// re-reads x.
#include "bitnet_device.hpp"
#include "bitnet_internal.hpp"

namespace bitnet {

constexpr int kActThreads = 256;
constexpr int kActWaves = kActThreads / kWave;
constexpr int kActMaxVec = 16;         // register-resident path: up to 16 x 16 bytes per thread (256 or 1024 threads)

__device__ inline int quantize_one(float v, float inv) { return (int)(int8_t)(quantize_bits(v, inv) & 0xFFu); }

template <int kWaves = kActWaves>
__device__ inline float block_max_nonneg(float v, float* sh) {
    v = wave_max_nonneg(v);
    if (kWaves == 1) return v;
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[wave] = v;
    __syncthreads();
    float m = sh[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, sh[w]);
    return m;
}

// ---- register-resident vector path ----------------------------------------------------------------
// fp32: a 16-byte load is 4 elements -> 4 int8 = one 32-bit store.
// bf16: a 16-byte load is 8 elements -> 8 int8 = one 64-bit store.
// kVecs 16-byte loads per thread hold the token (the launcher picks the smallest that covers K, which keeps the
// register count and with it the number of resident tokens per CU in proportion to K); 1024 threads for the rows
// 256 threads cannot hold.
// kAny: rows that start anywhere and need not fill their last load (K of any length, any base): the same loads and stores at
// element alignment, and the last K % kElems elements one each in the threads that come after the row's whole loads (in one thread
// they were up to seven loads and seven stores in a row: 30000 x 503 bf16 41 us, now 18; one element a thread throughout 28).
template <bool kBf16, int kVecs, int kThreads, bool kAny = false>
__global__ __launch_bounds__(kThreads) void quantize_acts_vec(const void* __restrict__ xv, int64_t K,
                                                              int8_t* __restrict__ xq, float* __restrict__ sx) {
    constexpr int kElems = kBf16 ? 8 : 4;
    const int rest = kAny ? (int)(K % kElems) : 0;
    __shared__ float sh[kThreads / kWave];
    const int64_t m = blockIdx.x;
    const int nvec = (int)(K / kElems);
    const uint4* row = reinterpret_cast<const uint4*>(static_cast<const char*>(xv) + m * K * (kBf16 ? 2 : 4));
    uint4 raw[kVecs];
    float amax = 0.0f;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const int idx = v * kThreads + threadIdx.x;
        raw[v] = make_uint4(0, 0, 0, 0);
        if (!kAny) {
            if (idx < nvec) raw[v] = row[idx];
        } else if (idx < nvec) {
            __builtin_memcpy(&raw[v], reinterpret_cast<const char*>(row) + (int64_t)idx * 16, 16);
        } else if (idx < nvec + rest) {
            const int64_t at = (int64_t)nvec * (kElems - 1) + idx;
            raw[v].x = kBf16 ? reinterpret_cast<const uint16_t*>(row)[at] : reinterpret_cast<const uint32_t*>(row)[at];
        }
    }
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const uint32_t u[4] = {raw[v].x, raw[v].y, raw[v].z, raw[v].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (kBf16) {
                amax = fmaxf(amax, fabsf(__uint_as_float(u[e] << 16)));
                amax = fmaxf(amax, fabsf(__uint_as_float(u[e] & 0xFFFF0000u)));
            } else {
                amax = fmaxf(amax, fabsf(__uint_as_float(u[e])));
            }
        }
    }
    amax = block_max_nonneg<kThreads / kWave>(amax, sh);
    const float s = fmaxf(amax, kEps);
    const float inv = kQb / s;                             // one IEEE division per token
    if (threadIdx.x == 0) sx[m] = s;

    int8_t* out = xq + m * K;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const int idx = v * kThreads + threadIdx.x;
        if (idx >= nvec + rest) continue;
        const uint32_t u[4] = {raw[v].x, raw[v].y, raw[v].z, raw[v].w};
        if (kAny) {
            uint32_t code[2];
            if (kBf16) {
                code[0] = pack4_quantized(__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u),
                                          __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xFFFF0000u), inv);
                code[1] = pack4_quantized(__uint_as_float(u[2] << 16), __uint_as_float(u[2] & 0xFFFF0000u),
                                          __uint_as_float(u[3] << 16), __uint_as_float(u[3] & 0xFFFF0000u), inv);
            } else {
                code[0] = pack4_quantized(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3]), inv);
                code[1] = 0;
            }
            if (idx < nvec) __builtin_memcpy(out + (int64_t)idx * kElems, code, kElems);
            else out[(int64_t)nvec * (kElems - 1) + idx] = (int8_t)code[0];
        } else if (kBf16) {
            const uint32_t lo = pack4_quantized(__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u),
                                                __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xFFFF0000u), inv);
            const uint32_t hi = pack4_quantized(__uint_as_float(u[2] << 16), __uint_as_float(u[2] & 0xFFFF0000u),
                                                __uint_as_float(u[3] << 16), __uint_as_float(u[3] & 0xFFFF0000u), inv);
            reinterpret_cast<uint2*>(out)[idx] = make_uint2(lo, hi);
        } else {
            reinterpret_cast<uint32_t*>(out)[idx] = pack4_quantized(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]),
                                                                    __uint_as_float(u[3]), inv);
        }
    }
}

// ---- any-shape path: two sweeps, element loads -----------------------------------------------------
template <bool kBf16>
__global__ __launch_bounds__(kActThreads) void quantize_acts_any(const void* __restrict__ xv, int64_t K,
                                                                 int8_t* __restrict__ xq, float* __restrict__ sx) {
    __shared__ float sh[kActWaves];
    const int64_t m = blockIdx.x;
    const float* rf = static_cast<const float*>(xv) + m * K;
    const uint16_t* rh = static_cast<const uint16_t*>(xv) + m * K;
    float amax = 0.0f;
    for (int64_t k = threadIdx.x; k < K; k += kActThreads)
        amax = fmaxf(amax, fabsf(kBf16 ? bf16_to_f32(rh[k]) : rf[k]));
    amax = block_max_nonneg(amax, sh);
    const float s = fmaxf(amax, kEps);
    const float inv = kQb / s;
    if (threadIdx.x == 0) sx[m] = s;
    int8_t* out = xq + m * K;
    for (int64_t k = threadIdx.x; k < K; k += kActThreads)
        out[k] = (int8_t)quantize_one(kBf16 ? bf16_to_f32(rh[k]) : rf[k], inv);
}

// ---------------------------------------------------------------------------------------------------
// Producers of int8 activations: the operations that precede a BitLinear layer in a LLaMA-style block
// (Section 2, "LLaMA-alike components": RMSNorm, SwiGLU) with the activation quantization fused in,
// so that the normalised / gated activations never travel through HBM as bf16.
// ---------------------------------------------------------------------------------------------------
constexpr int kProdMaxChunks = 16;     // register-resident path: up to 16 chunks of 4 elements per thread (256 or 1024 threads)

// four consecutive elements of a row, widened to fp32 (k is a multiple of 4; the row is 16- / 8-byte aligned)
template <bool kBf16>
__device__ inline void load_chunk(const void* row, int64_t k, float (&f)[4]) {
    if (kBf16) {
        const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(row) + k);
        f[0] = __uint_as_float(u.x << 16);
        f[1] = __uint_as_float(u.x & 0xFFFF0000u);
        f[2] = __uint_as_float(u.y << 16);
        f[3] = __uint_as_float(u.y & 0xFFFF0000u);
    } else {
        const float4 v = *reinterpret_cast<const float4*>(static_cast<const float*>(row) + k);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
}
template <bool kBf16>
__device__ inline float load_elem(const void* row, int64_t k) {
    return kBf16 ? bf16_to_f32(static_cast<const uint16_t*>(row)[k]) : static_cast<const float*>(row)[k];
}

__device__ inline uint32_t pack4(const float (&v)[4], float inv) { return pack4_quantized(v[0], v[1], v[2], v[3], inv); }

// one 16-byte piece of a row widened to fp32: eight bf16 or four fp32 elements
template <bool kBf16>
__device__ inline void expand_vec(const uint4& q, float (&f)[kBf16 ? 8 : 4]) {
    const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (kBf16) {
            f[2 * e] = __uint_as_float(u[e] << 16);
            f[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
        } else {
            f[e] = __uint_as_float(u[e]);
        }
    }
}

// r = (float)(1 / sqrt(mean(x^2) + eps)) from the threads' double-double partial sums of squares.  Every wave adds
// up its lanes; wave 0 alone then adds the waves, divides and takes the root in fp64 -- a hundred dependent
// instructions that the other waves' SIMDs can give to other tokens meanwhile -- and hands r over through LDS.
template <int kWaves>
__device__ inline float rms_scale(dd v, int64_t K, float eps, double* sh_hi, double* sh_lo, float* shr) {
    const dd w = wave_sum_dd(v);
    if (kWaves == 1) return (float)(1.0 / sqrt((w.hi + w.lo) / (double)K + (double)eps));
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sh_hi[wave] = w.hi; sh_lo[wave] = w.lo; }
    __syncthreads();
    if (wave == 0) {
        dd t{sh_hi[0], sh_lo[0]};
#pragma unroll
        for (int q = 1; q < kWaves; ++q) dd_add_dd(t, dd{sh_hi[q], sh_lo[q]});
        const double ms = (t.hi + t.lo) / (double)K;
        const float r = (float)(1.0 / sqrt(ms + (double)eps));
        if (threadIdx.x == 0) shr[0] = r;
    }
    __syncthreads();
    return shr[0];
}

// RMSNorm -> absmax int8.  Per token: ms = mean of squares (exact: squares of fp32 values are exact in
// fp64 and the sum is carried in double-double), r = (float)(1 / sqrt(ms + eps)) in fp64, z = (x * r) * g
// in fp32, then the per-token quantization of z.  r is the definition's float in every case, but the double-double sum, the
// division and the square root are only gone through where a plain fp64 sum leaves r open (rms_from_rounded_sum): 1 x 3200
// bf16 2.72 -> 2.17 us, 29 x 4096 3.10 -> 2.55, 2048 x 5120 11.7 -> 9.7, and 0.3 us off a decode launch with the norm in front.
//
// Register-resident form: the token is read once, kVecs 16-byte loads per thread (the launcher picks the smallest
// count that covers K), and stays in registers *as loaded* -- bf16 pairs are widened where they are used -- so that a
// workgroup needs few registers and a CU holds many tokens at different stages: a token is a load, a reduction, a
// load of the gain and another reduction in a row, and only tokens in other phases can hide one token's waits.  z is kept in
// registers between the absmax and the rounding where that takes at most 32 of them and recomputed with the same two
// multiplications otherwise.
template <bool kBf16, int kVecs, int kThreads, bool kGainFirst>
__global__ __launch_bounds__(kThreads) void rmsnorm_quantize_vec(
        const void* __restrict__ xv, const float* __restrict__ g, float eps, int64_t K, int8_t* __restrict__ xq,
        float* __restrict__ sx) {
    constexpr int kElems = kBf16 ? 8 : 4;
    constexpr int kWaves = kThreads / kWave;
    constexpr bool kKeepZ = kVecs * kElems <= 32;
    __shared__ double sh_hi[kWaves], sh_lo[kWaves];
    __shared__ float sh[kWaves + 1];                               // the waves' maxima; r of the token behind them
    const int64_t m = blockIdx.x;
    const int nvec = (int)(K / kElems);
    const uint4* row = reinterpret_cast<const uint4*>(static_cast<const char*>(xv) + m * K * (kBf16 ? 2 : 4));
    const float4* g4 = reinterpret_cast<const float4*>(g);
    uint4 raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const int idx = v * kThreads + threadIdx.x;
        raw[v] = make_uint4(0, 0, 0, 0);
        if (idx < nvec) raw[v] = row[idx];
    }
    // kGainFirst: the gain is requested with the token.  In a model every layer has its own, out of the caches by the time
    // the layer's turn comes, and a load that waits for the reduction adds its whole trip to the chain.
    float4 gk[kGainFirst ? kVecs * kElems / 4 : 1];
    if (kGainFirst && g) {
#pragma unroll
        for (int v = 0; v < kVecs; ++v)
#pragma unroll
            for (int q = 0; q < kElems / 4; ++q)
                gk[v * (kElems / 4) + q] = g4[min(v * kThreads + (int)threadIdx.x, nvec - 1) * (kElems / 4) + q];
    }

    // The mean of squares in plain fp64 (the squares are exact), four accumulators; vectors past the row hold zeros and are
    // skipped whole.  It decides r except for a token in half a million.
    double sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        if (v * kThreads >= nvec) continue;                     // uniform
        float f[kElems];
        expand_vec<kBf16>(raw[v], f);
#pragma unroll
        for (int e = 0; e < kElems; ++e) sq[e & 3] = __builtin_fma((double)f[e], (double)f[e], sq[e & 3]);
    }
    double S = wave_sum_f64((sq[0] + sq[1]) + (sq[2] + sq[3]));
    if (kWaves > 1) {
        if ((threadIdx.x & 63) == 0) sh_hi[threadIdx.x >> 6] = S;
        __syncthreads();
        S = sh_hi[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) S += sh_hi[w];
    }
    float r;
    if (__builtin_expect(!rms_from_rounded_sum(S, 1.0 / (double)K, eps, &r), 0)) {      // the same for all threads
        // four interleaved double-double accumulators: the sums are exact, so splitting them changes nothing but the length
        // of the dependent chain
        dd acc[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
        for (int v = 0; v < kVecs; ++v) {
            if (v * kThreads >= nvec) continue;                 // uniform
            float f[kElems];
            expand_vec<kBf16>(raw[v], f);
#pragma unroll
            for (int e = 0; e < kElems; ++e) dd_add_double(acc[e & 3], (double)f[e] * (double)f[e]);
        }
        dd_add_dd(acc[0], acc[1]);
        dd_add_dd(acc[2], acc[3]);
        dd_add_dd(acc[0], acc[2]);
        __syncthreads();                                        // the waves' sums have been read
        r = rms_scale<kWaves>(acc[0], K, eps, sh_hi, sh_lo, sh + kWaves);
    }

    // z = (x * r) * g of one vector; the gain comes from the caches (every token reads the same K floats)
    auto scaled = [&](int v, int idx, float (&z)[kElems]) {
        expand_vec<kBf16>(raw[v], z);
        float gl[kElems];
        if (g) {
#pragma unroll
            for (int q = 0; q < kElems / 4; ++q) {
                const float4 t = kGainFirst ? gk[v * (kElems / 4) + q] : g4[idx * (kElems / 4) + q];
                gl[4 * q] = t.x; gl[4 * q + 1] = t.y; gl[4 * q + 2] = t.z; gl[4 * q + 3] = t.w;
            }
        }
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
            z[e] = z[e] * r;
            if (g) z[e] = z[e] * gl[e];
        }
    };

    float zk[kKeepZ ? kVecs : 1][kElems];
    float amax = 0.0f;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const int idx = v * kThreads + threadIdx.x;
        if (v * kThreads >= nvec) continue;                     // uniform
        if (idx < nvec) {
            float z[kElems];
            scaled(v, idx, z);
#pragma unroll
            for (int e = 0; e < kElems; ++e) {
                amax = fmaxf(amax, fabsf(z[e]));
                if (kKeepZ) zk[v][e] = z[e];
            }
        }
    }
    amax = block_max_nonneg<kWaves>(amax, sh);
    const float s = fmaxf(amax, kEps);
    const float inv = kQb / s;
    if (threadIdx.x == 0) sx[m] = s;

    int8_t* out = xq + m * K;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
        const int idx = v * kThreads + threadIdx.x;
        if (v * kThreads >= nvec) continue;                     // uniform
        if (idx >= nvec) continue;
        float z[kElems];
        if (kKeepZ) {
#pragma unroll
            for (int e = 0; e < kElems; ++e) z[e] = zk[v][e];
        } else {
            scaled(v, idx, z);                                  // the same two multiplications: the same z
        }
        if (kBf16) {
            reinterpret_cast<uint2*>(out)[idx] = make_uint2(pack4_quantized(z[0], z[1], z[2], z[3], inv),
                                                            pack4_quantized(z[4], z[5], z[6], z[7], inv));
        } else {
            reinterpret_cast<uint32_t*>(out)[idx] = pack4_quantized(z[0], z[1], z[2], z[3], inv);
        }
    }
}

// Any K and any alignment: three sweeps over the token in memory, element loads.
template <bool kBf16, int kThreads>
__global__ __launch_bounds__(kThreads) void rmsnorm_quantize_any(
        const void* __restrict__ xv, const float* __restrict__ g, float eps, int64_t K, int8_t* __restrict__ xq,
        float* __restrict__ sx) {
    constexpr int kWaves = kThreads / kWave;
    __shared__ double sh_hi[kWaves], sh_lo[kWaves];
    __shared__ float sh[kWaves + 1];                               // the waves' maxima; r of the token behind them
    const int64_t m = blockIdx.x;
    const void* row = static_cast<const char*>(xv) + m * K * (kBf16 ? 2 : 4);
    int8_t* out = xq + m * K;
    dd acc{0.0, 0.0};
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        const double a = (double)load_elem<kBf16>(row, k);
        dd_add_double(acc, a * a);
    }
    const float r = rms_scale<kWaves>(acc, K, eps, sh_hi, sh_lo, sh + kWaves);
    float amax = 0.0f;
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        float z = load_elem<kBf16>(row, k) * r;
        if (g) z = z * g[k];
        amax = fmaxf(amax, fabsf(z));
    }
    amax = block_max_nonneg<kWaves>(amax, sh);
    const float s = fmaxf(amax, kEps);
    const float inv = kQb / s;
    if (threadIdx.x == 0) sx[m] = s;
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        float z = load_elem<kBf16>(row, k) * r;                    // the same two multiplies: the same z
        if (g) z = z * g[k];
        out[k] = (int8_t)quantize_one(z, inv);
    }
}

// SwiGLU gating -> absmax int8.  gu is [M][2F]: h = silu(gu[:, :F]) * gu[:, F:], then the per-token
// quantization of h.
template <bool kBf16, int kChunks, int kThreads>
__global__ __launch_bounds__(kThreads) void swiglu_quantize_kernel(
        const void* __restrict__ guv, int64_t F, int8_t* __restrict__ hq, float* __restrict__ sh_out) {
    constexpr int kWaves = kThreads / kWave;
    constexpr bool kVec = kChunks > 0;                             // as for rmsnorm_quantize_kernel
    __shared__ float sh[kWaves];
    const int64_t m = blockIdx.x;
    const void* gate = static_cast<const char*>(guv) + m * 2 * F * (kBf16 ? 2 : 4);
    const void* up = static_cast<const char*>(gate) + F * (kBf16 ? 2 : 4);
    int8_t* out = hq + m * F;
    const int nchunks = (int)(F / 4);
    float v[kVec ? kChunks : 1][4];

    float amax = 0.0f;
    if (kVec) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            if (i * kThreads >= nchunks) continue;              // uniform: whole iterations past the row
            const int c = i * kThreads + threadIdx.x;
            if (c < nchunks) {
                float a[4], b[4];
                load_chunk<kBf16>(gate, 4 * (int64_t)c, a);
                load_chunk<kBf16>(up, 4 * (int64_t)c, b);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[i][e] = swiglu_one(a[e], b[e]);
                    amax = fmaxf(amax, fabsf(v[i][e]));
                }
            }
        }
    } else {
        for (int64_t f = threadIdx.x; f < F; f += kThreads)
            amax = fmaxf(amax, fabsf(swiglu_one(load_elem<kBf16>(gate, f), load_elem<kBf16>(up, f))));
    }
    amax = block_max_nonneg<kWaves>(amax, sh);
    const float s = fmaxf(amax, kEps);
    const float inv = kQb / s;
    if (threadIdx.x == 0) sh_out[m] = s;

    if (kVec) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            if (i * kThreads >= nchunks) continue;              // uniform: whole iterations past the row
            const int c = i * kThreads + threadIdx.x;
            if (c < nchunks) reinterpret_cast<uint32_t*>(out)[c] = pack4(v[i], inv);
        }
    } else {
        for (int64_t f = threadIdx.x; f < F; f += kThreads)
            out[f] = (int8_t)quantize_one(swiglu_one(load_elem<kBf16>(gate, f), load_elem<kBf16>(up, f)), inv);
    }
}

// The same for bf16 rows.  The gate costs ~45 VALU instructions an element (exponential, IEEE division): more time than the bytes.
// But silu's argument is a bf16 value, so a workgroup holds it for every value of magnitude 2^-15 ... 2^8 (23 exponents x 128
// mantissas x 2 signs, 23 KB of LDS: the very same function, the same bits) and looks it up for all elements of all its tokens.
// kCopy: the table is a constant array, made by the compiler with the steps of silu_one, and comes to LDS beside the first token;
// evaluating it is 1.8 us in front of that token, which is all a workgroup has where tokens are few (7B stack at 29 tokens 323.8 ->
// 320.7 us).  Many workgroups evaluate it instead: they would all read the same 23 KB at once.
// Zero has an entry too -- a projection's integer sum is 0 for one output in a thousand,
// which is one in half of all wave-wide vectors -- and a wave that holds any other magnitude goes through silu_beyond_table.  A
// workgroup walks tokens blockIdx.x, + workgroups, ... with the next token's loads in flight under the current one's work.
// bf16, alone, arithmetic / table: 64 x 11008 4.8 / 4.5 us, 8 x 14336 5.2 / 4.1, 2048 x 13824 38.5 / 25.4, 4096 x 28672 134 / 113
// (5.2 TB/s, what a device copy reaches).  Gates that are all beyond the table (around 1e4, or 1e-5), table evaluated: 64 x 11008 6.0,
// 2048 x 13824 31.3, 4096 x 28672 126.
constexpr int kSiluBase = (127 - 15) << 7;                 // bf16 bits of 2^-15
constexpr int kSiluLimit = (127 + 8) << 7;                 // ... and of 2^8
constexpr int kSiluSpan = kSiluLimit - kSiluBase + 1;      // zero, and the magnitudes in between

// silu of any bf16 value, with the table's help: the bits of silu_one, checked for every one of the 65536.  From 88 on
// exp32(-gate) is one constant for each sign, and silu a multiple of the gate: the entry of the same mantissa in [2^7, 2^8)
// times a power of two.  Below 2^-15 the exponential's polynomial comes down to its last three terms, and the divisor is so
// close to 2 that a quotient from the first term of a series needs one correction.
__device__ inline float silu_beyond_table(uint32_t bits, const float* table) {
    const float g = __uint_as_float(bits << 16);
    const uint32_t mag = bits & 0x7FFFu, sign = bits >> 15;
    const bool high = mag >= (uint32_t)kSiluLimit;
    const uint32_t at = high ? (uint32_t)(kSiluLimit - 128) | (mag & 127u) : mag;
    const uint32_t d = at < (uint32_t)kSiluBase ? 0u : at - (uint32_t)(kSiluBase - 1);
    float v = table[2 * d + sign] * (high ? __uint_as_float(((mag >> 7) - 7u) << 23) : 1.0f);
    const float s = 1.0f + __builtin_fmaf(-g, __builtin_fmaf(g, -0.5f, 1.0f), 1.0f);
    const float q = __builtin_fmaf(0.5f * g, __builtin_fmaf(s, -0.5f, 1.0f), 0.5f * g);     // g / s by a term of its series ...
    if (mag - 1u < (uint32_t)(kSiluBase - 1))              // ... and the remainder over barely less than 2
        v = __builtin_fmaf(__builtin_fmaf(-q, s, g), 0x1.000002p-1f, q);
    if (mag >= 0x7F80u) v = g;                             // infinities keep their sign, NaN stays
    return v;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// [0: zero, k: the magnitude of bits kSiluBase + k - 1][sign]
constexpr int kSiluEntries = (2 * kSiluSpan + 3) & ~3;
struct SiluTable { float v[kSiluEntries]; };
constexpr float silu_of_bits(uint32_t bits) {              // silu_one, step by step
    const float gate = __builtin_bit_cast(float, bits << 16);
    float t = -gate;
    t = t < -87.0f ? -87.0f : t > 88.0f ? 88.0f : t;
    const float n = (t * 1.44269504f + kRoundMagic) - kRoundMagic;          // rint
    float r = t - n * 0.693359375f;
    r = r - n * -2.12194440e-4f;
    float p = 1.0f / 720.0f;
    p = p * r + 1.0f / 120.0f;
    p = p * r + 1.0f / 24.0f;
    p = p * r + 1.0f / 6.0f;
    p = p * r + 0.5f;
    p = p * r + 1.0f;
    p = p * r + 1.0f;
    return gate / (1.0f + p * __builtin_bit_cast(float, (uint32_t)(127 + (int)n) << 23));      // n is within -126 ... 127
}
constexpr SiluTable silu_table() {
    SiluTable t{};
    for (int i = 0; i < 2 * kSiluSpan; ++i)
        t.v[i] = silu_of_bits((uint32_t)(i < 2 ? 0 : kSiluBase - 1 + (i >> 1)) | (uint32_t)(i & 1) << 15);
    return t;
}
__device__ constexpr SiluTable kSiluTable = silu_table();

template <int kVecs, int kThreads, bool kCopy>
__global__ __launch_bounds__(kThreads) void swiglu_quantize_table(const uint16_t* __restrict__ gu, int64_t M, int64_t F,
                                                                  int8_t* __restrict__ hq, float* __restrict__ sh_out, int workgroups) {
    constexpr int kWaves = kThreads / kWave;
    __shared__ __attribute__((aligned(16))) float table[kSiluEntries];
    __shared__ float sh[2][kWaves];
    const int nvec = (int)(F / 8);
    uint4 g[kVecs], u[kVecs];
    auto request = [&](int64_t m) {
        const uint4* gate = reinterpret_cast<const uint4*>(gu + m * 2 * F);
#pragma unroll
        for (int v = 0; v < kVecs; ++v) {
            const int idx = v * kThreads + threadIdx.x;
            g[v] = u[v] = make_uint4(0, 0, 0, 0);
            if (idx < nvec) { g[v] = gate[idx]; u[v] = gate[nvec + idx]; }
        }
    };
    int64_t m = blockIdx.x;
    request(m);
    if (kCopy) {
        constexpr int kCopies = (kSiluEntries / 4 + kThreads - 1) / kThreads;
        float4 part[kCopies];
#pragma unroll
        for (int c = 0; c < kCopies; ++c) part[c] = reinterpret_cast<const float4*>(kSiluTable.v)[min(c * kThreads + (int)threadIdx.x, kSiluEntries / 4 - 1)];
#pragma unroll
        for (int c = 0; c < kCopies; ++c)
            if (c * kThreads + (int)threadIdx.x < kSiluEntries / 4) reinterpret_cast<float4*>(table)[c * kThreads + threadIdx.x] = part[c];
    } else {
        for (int i = threadIdx.x; i < 2 * kSiluSpan; i += kThreads)
            table[i] = silu_one(bf16_to_f32((uint16_t)((i < 2 ? 0 : kSiluBase - 1 + (i >> 1)) | ((i & 1) << 15))));
    }
    __syncthreads();

    for (int parity = 0; m < M; parity ^= 1) {
        uint4 cg[kVecs], cu[kVecs];
#pragma unroll
        for (int v = 0; v < kVecs; ++v) { cg[v] = g[v]; cu[v] = u[v]; }
        const int64_t next = m + workgroups;
        if (next < M) request(next);
        float h[kVecs][8];
        float amax = 0.0f;
#pragma unroll
        for (int v = 0; v < kVecs; ++v) {
            if (v * kThreads + (int)threadIdx.x >= nvec) continue;
            const uint32_t gw[4] = {cg[v].x, cg[v].y, cg[v].z, cg[v].w}, uw[4] = {cu[v].x, cu[v].y, cu[v].z, cu[v].w};
            constexpr unsigned short kLow = kSiluBase - 1;
            u16x2 d[4], top = {0, 0}, low = {0xFFFF, 0xFFFF};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u16x2 mag = __builtin_bit_cast(u16x2, gw[e] & 0x7FFF7FFFu);
                d[e] = __builtin_elementwise_sub_sat(mag, (u16x2){kLow, kLow});
                top = __builtin_elementwise_max(top, d[e]);
                low = __builtin_elementwise_min(low, mag - (u16x2){1, 1});        // zero wraps: it is no low magnitude
            }
            const bool inside = (top.x > top.y ? top.x : top.y) < kSiluSpan && (low.x < low.y ? low.x : low.y) >= kLow;
            if (__builtin_expect(!__any(!inside), 1)) {             // the same for the wave
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t at = (__builtin_bit_cast(uint32_t, d[e]) << 1) | ((gw[e] >> 15) & 0x00010001u);
                    h[v][2 * e] = table[at & 0xFFFFu];
                    h[v][2 * e + 1] = table[at >> 16];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    h[v][2 * e] = silu_beyond_table(gw[e] & 0xFFFFu, table);
                    h[v][2 * e + 1] = silu_beyond_table(gw[e] >> 16, table);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                h[v][2 * e] *= __uint_as_float(uw[e] << 16);
                h[v][2 * e + 1] *= __uint_as_float(uw[e] & 0xFFFF0000u);
                amax = fmaxf(amax, fmaxf(fabsf(h[v][2 * e]), fabsf(h[v][2 * e + 1])));
            }
        }
        amax = block_max_nonneg<kWaves>(amax, sh[parity]);     // two buffers: one barrier per token
        const float s = fmaxf(amax, kEps);
        const float inv = kQb / s;
        if (threadIdx.x == 0) sh_out[m] = s;
        uint2* out = reinterpret_cast<uint2*>(hq + m * F);
#pragma unroll
        for (int v = 0; v < kVecs; ++v) {
            const int idx = v * kThreads + threadIdx.x;
            if (idx < nvec) out[idx] = make_uint2(pack4_quantized(h[v][0], h[v][1], h[v][2], h[v][3], inv), pack4_quantized(h[v][4], h[v][5], h[v][6], h[v][7], inv));
        }
        m = next;
    }
}

// SwiGLU, threads per token.  Few tokens: 1024, so that the dependent chains of the gate (exponential, division) interleave over
// four waves per SIMD; many: 256, and the tokens fill the CUs.  From 64 to 1023 tokens it is the row that decides: with 1024 threads
// the chip runs fewer tokens at a time, which pays while the row gives all of them work (fp32, 256 threads / 1024: 100 x 8640 9.6 /
// 5.1 us, 600 x 11008 17.2 / 15.2, 1000 x 4096 9.2 / 8.8; bf16: 500 x 1536 3.6 / 3.4, 800 x 2560 5.5 / 5.3) and not on narrow rows (bf16,
// 600 x 264 2.7 / 3.4, 1000 x 1024 3.6 / 4.3).  The sweeping form, whose chains are longer, from half as wide a row on (fp32, 600 x
// 1001 4.9 / 4.6, 800 x 1001 5.2 / 5.4).  Rows too long for 256 threads' registers take 1024 at any token count.
static bool producer_wide(bool vec, int64_t M, int64_t cols) {
    if (M < 64 || cols > (int64_t)kProdMaxChunks * 256 * 4) return true;
    return M < 1024 && (vec ? cols > 1024 && cols >= 3 * M : cols > 256 && 2 * cols >= 3 * M);
}

// chunks of four: rows must start on a chunk boundary of the input loads and of the 32-bit stores
static bool producer_vec_ok(const void* in, size_t esz, int64_t cols, const void* out) {
    return cols % 4 == 0 && cols <= (int64_t)kProdMaxChunks * 1024 * 4 &&
           reinterpret_cast<uintptr_t>(in) % (4 * esz) == 0 && reinterpret_cast<uintptr_t>(out) % 4 == 0;
}

// threads per token and register chunks per thread for a row of `cols` elements (chunks == 0: the sweeping form)
static void producer_shape(bool vec, int64_t M, int64_t cols, int* threads, int* chunks) {
    *threads = producer_wide(vec, M, cols) ? 1024 : 256;
    *chunks = 0;
    if (!vec) return;
    const int64_t need = ceil_div(cols, (int64_t)*threads * 4);
    *chunks = need <= 4 ? 4 : need <= 8 ? 8 : 16;
}

#define PRODUCER_PICK(B_)                                                                                        \
    do {                                                                                                         \
        if (threads == 1024) {                                                                                   \
            if (chunks == 4) GO(B_, 4, 1024); else if (chunks == 8) GO(B_, 8, 1024);                             \
            else if (chunks == 16) GO(B_, 16, 1024); else GO(B_, 0, 1024);                                       \
        } else {                                                                                                 \
            if (chunks == 4) GO(B_, 4, 256); else if (chunks == 8) GO(B_, 8, 256);                               \
            else if (chunks == 16) GO(B_, 16, 256); else GO(B_, 0, 256);                                         \
        }                                                                                                        \
    } while (0)

// A workgroup per token and up to 1024 threads in it: tokens beyond what a launch has threads for come in further launches.
constexpr int64_t kTokenSlab = kMaxGridThreads / 1024 / 2;
template <typename Launch>
static hipError_t in_token_slabs(int64_t M, Launch&& launch) {
    for (int64_t m0 = 0; m0 < M; m0 += kTokenSlab) {
        const hipError_t e = launch(m0, M - m0 < kTokenSlab ? M - m0 : kTokenSlab);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_rmsnorm_quantize(const void* x, bool bf16, const float* g, float eps, int64_t M, int64_t K,
                                   int8_t* xq, float* sx, hipStream_t stream) {
    if (M > kTokenSlab)
        return in_token_slabs(M, [&](int64_t m0, int64_t n) {
            return launch_rmsnorm_quantize(static_cast<const char*>(x) + m0 * K * (bf16 ? 2 : 4), bf16, g, eps, n, K, xq + m0 * K, sx + m0, stream);
        });
    const int elems = bf16 ? 8 : 4;
    const int max_vecs = bf16 ? 8 : 16;                            // 64 token elements per thread at most
    const bool aligned = K % elems == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
                         reinterpret_cast<uintptr_t>(xq) % (bf16 ? 8 : 4) == 0 && reinterpret_cast<uintptr_t>(g) % 16 == 0;
    const int64_t nvec = K / elems;
    // 256 threads while four loads each hold the token: the reductions over sixteen waves cost a workgroup of 1024 more than
    // its shorter chains of the exact sum save (bf16, 256 / 1024 threads: 1 x 3200 2.95 / 3.68 us, 29 x 4096 3.33 / 4.12,
    // 60 x 8192 4.63 / 4.77, 200 x 2048 3.2 / 4.1).  Longer rows of few tokens: 1024 (1 x 14336 6.58 / 4.78), of many tokens
    // 256, and the tokens fill the CUs (one or two waves per token were measured too: slower at every size from 64 to 4096
    // tokens); rows that would need more than eight loads per thread at 256 threads take 1024 at any count (sixteen loads
    // cost occupancy: fp32 rows of 13824 run 5-15 % faster on 1024 threads)
    const int threads = (nvec > (int64_t)8 * 256 || (M < 64 && nvec > (int64_t)4 * 256)) ? 1024 : 256;
    const int64_t need = ceil_div(nvec, threads);
    dim3 grid((unsigned)M), block(threads);
    // up to a token per CU: nothing else there hides a load behind the reduction, and no one needs the registers (7B stack at 29
    // tokens, eight layers, 364.5 -> 356 us; 200 x 4096 with the product behind it 19.9 -> 19.5; no difference from 400 tokens on)
    const bool first = M <= 256;
#define GO(B_, V_, T_)                                                                                           \
    do {                                                                                                         \
        if constexpr (V_ * (B_ ? 8 : 4) <= 32) {                                                                 \
            if (first) { hipLaunchKernelGGL((rmsnorm_quantize_vec<B_, V_, T_, true>), grid, block, 0, stream, x, g, eps, K, xq, sx); break; } \
        }                                                                                                        \
        hipLaunchKernelGGL((rmsnorm_quantize_vec<B_, V_, T_, false>), grid, block, 0, stream, x, g, eps, K, xq, sx); \
    } while (0)
#define PICK(B_, T_)                                                                                             \
    do {                                                                                                         \
        if (need <= 1) GO(B_, 1, T_); else if (need <= 2) GO(B_, 2, T_); else if (need <= 4) GO(B_, 4, T_);      \
        else if (need <= 8) GO(B_, 8, T_); else if (!B_ && T_ == 1024) GO(false, 16, 1024);                      \
    } while (0)
    if (aligned && need <= max_vecs) {
        if (bf16) { if (threads == 1024) PICK(true, 1024); else PICK(true, 256); }
        else      { if (threads == 1024) PICK(false, 1024); else PICK(false, 256); }
    } else {
        if (bf16) {
            if (threads >= 1024) hipLaunchKernelGGL((rmsnorm_quantize_any<true, 1024>), grid, block, 0, stream, x, g, eps, K, xq, sx);
            else                 hipLaunchKernelGGL((rmsnorm_quantize_any<true, 256>), grid, block, 0, stream, x, g, eps, K, xq, sx);
        } else {
            if (threads >= 1024) hipLaunchKernelGGL((rmsnorm_quantize_any<false, 1024>), grid, block, 0, stream, x, g, eps, K, xq, sx);
            else                 hipLaunchKernelGGL((rmsnorm_quantize_any<false, 256>), grid, block, 0, stream, x, g, eps, K, xq, sx);
        }
    }
#undef GO
#undef PICK
    return hipGetLastError();
}

// Where the table form is the faster one, us, arithmetic / table: alone, 1 x 11008 4.2 / 3.5, 8 x 14336 5.2 / 4.1, 29 x 11008 4.7 / 4.3,
// 29 x 8192 3.9 / 3.9, 128 x 5504 3.5 / 4.0, 256 x 4096 3.4 / 4.1; measured where the launch stands in use (behind the gate/up
// product and in front of the down product, all of it) 5120 -> 13824 at 128 tokens, two layers, 179.3 / 176.2, at 1024 201.8 /
// 194.2; 2048 tokens 356 / 345.  Narrow rows leave most of the 1024 threads idle and pay for the table all the same: 700 x 4096
// 33.6 / 34.2, 64 x 5504 equal.
static bool swiglu_by_table(const void* gu, int64_t M, int64_t F, const void* hq) {
    if (F % 8 != 0 || F > 32768 || reinterpret_cast<uintptr_t>(gu) % 16 != 0 || reinterpret_cast<uintptr_t>(hq) % 8 != 0) return false;
    return F >= 5120 && M >= (F >= 9216 ? 1 : F >= 8192 ? 64 : 256);
}

hipError_t launch_swiglu_quantize(const void* gu, bool bf16, int64_t M, int64_t F, int8_t* hq, float* sh,
                                  hipStream_t stream) {
    if (M > kTokenSlab)
        return in_token_slabs(M, [&](int64_t m0, int64_t n) {
            return launch_swiglu_quantize(static_cast<const char*>(gu) + m0 * 2 * F * (bf16 ? 2 : 4), bf16, n, F, hq + m0 * F, sh + m0, stream);
        });
    if (bf16 && swiglu_by_table(gu, M, F, hq)) {
        const uint16_t* in = static_cast<const uint16_t*>(gu);
        const int wgs = (int)(M < 256 ? M : 256);          // one per CU: two and four were no faster
        // The constant array until so many workgroups read it that evaluating it costs less (us, copied / evaluated: 29 x 11008
        // 4.3 / 4.9, 128 x 11008 4.8 / 5.1, 29 x 28672 6.5 / 6.7; 128 x 14336 5.7 / 5.5, 64 x 28672 7.9 / 7.4, 256 x 11008 6.2 / 5.5)
        const bool copy = M * F <= (int64_t)3 << 19;
#define TABLE(V_)                                                                                                \
    do {                                                                                                         \
        if (copy) hipLaunchKernelGGL((swiglu_quantize_table<V_, 1024, true>), dim3((unsigned)wgs), dim3(1024), 0, stream, in, M, F, hq, sh, wgs); \
        else hipLaunchKernelGGL((swiglu_quantize_table<V_, 1024, false>), dim3((unsigned)wgs), dim3(1024), 0, stream, in, M, F, hq, sh, wgs); \
    } while (0)
        if (F <= 8192) TABLE(1);
        else if (F <= 16384) TABLE(2);
        else TABLE(4);
#undef TABLE
        return hipGetLastError();
    }
    int threads, chunks;
    producer_shape(producer_vec_ok(gu, bf16 ? 2 : 4, F, hq), M, F, &threads, &chunks);
    dim3 grid((unsigned)M), block(threads);
#define GO(B_, C_, T_) hipLaunchKernelGGL((swiglu_quantize_kernel<B_, C_, T_>), grid, block, 0, stream, gu, F, hq, sh)
    if (bf16) PRODUCER_PICK(true); else PRODUCER_PICK(false);
#undef GO
    return hipGetLastError();
}
#undef PRODUCER_PICK

hipError_t launch_quantize_acts(const void* x, bool bf16, int64_t M, int64_t K, int8_t* xq, float* sx,
                                hipStream_t stream) {
    if (M > kTokenSlab)
        return in_token_slabs(M, [&](int64_t m0, int64_t n) {
            return launch_quantize_acts(static_cast<const char*>(x) + m0 * K * (bf16 ? 2 : 4), bf16, n, K, xq + m0 * K, sx + m0, stream);
        });
    const int elems = bf16 ? 8 : 4;
    const bool aligned = (reinterpret_cast<uintptr_t>(x) % 16 == 0) && (K % elems == 0) &&
                         (reinterpret_cast<uintptr_t>(xq) % 8 == 0);
    const int64_t nvec = K / elems;
    const int threads = nvec <= (int64_t)kActMaxVec * kActThreads ? kActThreads : 1024;
    const int64_t need = ceil_div(nvec, threads);
    dim3 grid((unsigned)M), block(threads);
#define GO(B_, V_, T_) hipLaunchKernelGGL((quantize_acts_vec<B_, V_, T_>), grid, block, 0, stream, x, K, xq, sx)
#define PICK(B_)                                                                                                 \
    do {                                                                                                         \
        if (threads == 1024) { if (need <= 8) GO(B_, 8, 1024); else if (!B_) GO(false, 16, 1024); }              \
        else if (need <= 2) GO(B_, 2, kActThreads);                                                              \
        else if (need <= 4) GO(B_, 4, kActThreads);                                                              \
        else if (need <= 8) GO(B_, 8, kActThreads);                                                              \
        else GO(B_, 16, kActThreads);                                                                            \
    } while (0)
    // (bf16 at 1024 threads and 16 loads per thread would spill: such rows, beyond 65536 elements, sweep instead)
    if (aligned && need <= ((threads == 1024 && bf16) ? 8 : kActMaxVec)) {
        if (bf16) PICK(true); else PICK(false);
    } else if (nvec < 8 * kActThreads && K * (bf16 ? 2 : 4) >= 256 && reinterpret_cast<uintptr_t>(x) % (bf16 ? 2 : 4) == 0) {
        // rows of any length and alignment that 256 threads hold in eight loads each (a ninth only for the last elements)
        // (200 x 3333 fp32, its product behind it: 20.4 us with element loads in two sweeps, 18.0).  Rows of less than 256 bytes are
        // done sooner by a thread per element (bf16, 8192 x 33 4.7 us, in loads of eight elements 5.6; 8192 x 129 6.4 / 6.1)
        block = dim3(kActThreads);
        const int64_t slots = nvec + K % elems;
#define ANY(B_, V_) hipLaunchKernelGGL((quantize_acts_vec<B_, V_, kActThreads, true>), grid, block, 0, stream, x, K, xq, sx)
#define PICK_ANY(B_) do { if (slots <= 2 * kActThreads) ANY(B_, 2); else if (slots <= 8 * kActThreads) ANY(B_, 8); else ANY(B_, 9); } while (0)
        if (bf16) PICK_ANY(true); else PICK_ANY(false);
#undef PICK_ANY
#undef ANY
    } else {
        block = dim3(kActThreads);
        if (bf16) hipLaunchKernelGGL(quantize_acts_any<true>, grid, block, 0, stream, x, K, xq, sx);
        else      hipLaunchKernelGGL(quantize_acts_any<false>, grid, block, 0, stream, x, K, xq, sx);
    }
#undef GO
#undef PICK
    return hipGetLastError();
}

}  // namespace bitnet
