// The 5-trits-per-byte format (1.6 bits per weight; the paper notes that 2 bits leave room above the
// 1.58-bit information content of a ternary weight, Section 3 of arXiv 2402.17764): unpack helper,
// reference product, weight-streaming kernels for M <= 16 and the passes between the two formats.
//
// Layout (bitnet.h): byte p of a 16-byte quad carries digits 0..3 = four consecutive columns 4p..4p+3
// and digit 4 = column 64 + p of the quad's 80 columns.  The streaming kernel keeps a 243-entry table
// in LDS that maps a byte to its five decoded operand bytes (64 * code), so a byte's first four digits
// arrive as one ready MFMA operand register; the sixteen fifth digits of a quad are gathered into the
// four registers of a fifth MFMA.  One step = 320 columns = five v_mfma_i32_16x16x64_i8 per row block.
#include "bitnet_device.hpp"
#include "bitnet_internal.hpp"
#include "gemv_common.hpp"

namespace bitnet {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kTritCols = 80;            // columns per quad

// byte offset and digit of column k of row n
__host__ __device__ inline void trit5_locate(int64_t n, int64_t k, int64_t RB, int64_t* byte_index, int* digit) {
    const int64_t s = k / kTritStep;
    const int c = (int)(k % kTritStep);
    const int g = c / kTritCols, q = c % kTritCols;
    const int64_t quad = 64 * (RB * s + (n >> 4)) + 16 * g + (n & 15);
    if (q < 64) { *byte_index = quad * 16 + (q >> 2); *digit = q & 3; }
    else        { *byte_index = quad * 16 + (q - 64); *digit = 4; }
}

__device__ inline int trit5_digit(uint32_t byte, int d) {
    const uint32_t p3 = d == 0 ? 1u : d == 1 ? 3u : d == 2 ? 9u : d == 3 ? 27u : 81u;
    return (int)((byte / p3) % 3u) - 1;
}

// chunks (16 rows x 320 columns, a wave each) of one repacking launch: half the threads that a grid dimension holds
constexpr int64_t kLaunchChunks = (int64_t)1 << 25;

// ---------------------------------------------------------------------------------------------------
// unpack helper and reference product
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void unpack_trit5(const uint8_t* __restrict__ packed, int64_t N, int64_t K, int64_t RB,
                                                    int8_t* __restrict__ codes) {
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < N * K; idx += (int64_t)gridDim.x * 256) {
        int64_t bi; int dg;
        trit5_locate(idx / K, idx % K, RB, &bi, &dg);
        codes[idx] = (int8_t)trit5_digit(packed[bi], dg);
    }
}

__global__ __launch_bounds__(256) void linear_reference_trit5(const int8_t* __restrict__ xq, const float* __restrict__ sx,
                                                              const uint8_t* __restrict__ packed,
                                                              const float* __restrict__ gamma, int64_t N, int64_t K,
                                                              int64_t RB, void* __restrict__ y, OutType yt) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t m = blockIdx.y;
    if (n >= N) return;
    const int8_t* xr = xq + m * K;
    int32_t acc = 0;
    for (int64_t k = 0; k < K; ++k) {
        int64_t bi; int dg;
        trit5_locate(n, k, RB, &bi, &dg);
        const int code = trit5_digit(packed[bi], dg);
        if (code > 0) acc += xr[k];
        else if (code < 0) acc -= xr[k];
    }
    const int64_t idx = m * N + n;
    if (yt == OutType::I32) static_cast<int32_t*>(y)[idx] = acc;
    else {
        const float v = (float)acc * ((gamma[0] * sx[m]) / kQb);
        if (yt == OutType::F32) static_cast<float*>(y)[idx] = v;
        else static_cast<uint16_t*>(y)[idx] = f32_to_bf16(v);
    }
}

// ---------------------------------------------------------------------------------------------------
// weight-streaming kernel, M <= 16
// ---------------------------------------------------------------------------------------------------
__device__ inline v4i trit_as_v4i(const uint4& u) {
    v4i a;
    a.x = (int)u.x; a.y = (int)u.y; a.z = (int)u.z; a.w = (int)u.w;
    return a;
}

// kR row blocks per wave, kS waves splitting K, kD steps of loads in flight (same scheme as the 2-bit kernel:
// branch-free masked loop, out-of-range steps / rows / tokens redirected and zeroed)
// Four waves per SIMD by declaration: with 129 registers the form with three steps in flight lost one of them.
template <int kR, int kS, int kD>
__global__ __launch_bounds__(kS * kWave, 4) void linear_gemv16_trit5(
        const int8_t* __restrict__ xq, const uint4* __restrict__ packed, const float* __restrict__ gamma, const float* __restrict__ sx,
        void* __restrict__ y, int N32, int K32, uint32_t flags /* tokens, output type */) {
    const int64_t K = K32, N = N32;
    const int M = flags_number(flags), RB = (int)((N + kRowsPerBlock - 1) / kRowsPerBlock), steps = (K32 + kTritStep - 1) / kTritStep;
    const int items = ((steps + kS - 1) / kS + kD - 1) / kD * kD;
    const OutType yt = flags_out_type(flags);
    __shared__ uint2 lut[256];                       // byte -> {digits 0..3 as 4 operand bytes, digit 4 as 1 byte}
    __shared__ v4i fold[kS][kR][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int rb0 = blockIdx.x * kR;

    for (int b = threadIdx.x; b < 256; b += kS * kWave) {
        uint32_t lo = 0, hi = 0;
        if (b < 243) {
#pragma unroll
            for (int dgt = 0; dgt < 4; ++dgt) lo |= ((uint32_t)(trit5_digit(b, dgt) * 64) & 0xFFu) << (8 * dgt);
            hi = (uint32_t)(trit5_digit(b, 4) * 64) & 0xFFu;
        }
        lut[b] = make_uint2(lo, hi);
    }

    const int64_t wstride = (int64_t)RB * 64;
    const uint4* wp[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) wp[a] = packed + (int64_t)min(rb0 + a, RB - 1) * 64 + lane;
    const int8_t* xg = xq + (int64_t)min(r, M - 1) * K;

    v4i acc[kR];
#pragma unroll
    for (int a = 0; a < kR; ++a) acc[a] = (v4i){0, 0, 0, 0};

    struct Stage { uint4 w[kR]; uint4 x[5]; };
    auto load = [&](Stage& s, int item) {
        const int sl = min(wave + item * kS, steps - 1);
#pragma unroll
        for (int a = 0; a < kR; ++a) s.w[a] = load_streaming_b128(wp[a] + (int64_t)sl * wstride);
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const int64_t col = min((int64_t)sl * kTritStep + kTritCols * g + 16 * j, K - 16);   // past K: zero codes
            s.x[j] = *reinterpret_cast<const uint4*>(xg + col);
        }
    };
    auto mac = [&](Stage& s, int item) {
        const bool live = wave + item * kS < steps;
#pragma unroll
        for (int a = 0; a < kR; ++a) {
            const uint32_t wd[4] = {s.w[a].x, s.w[a].y, s.w[a].z, s.w[a].w};
            v4i op[5];
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                // byte 121 = digits (1,1,1,1,1) = five zero codes: what a step past the end contributes
                const uint32_t byte = live ? ((wd[p >> 2] >> (8 * (p & 3))) & 0xFFu) : 121u;
                const uint2 e = lut[byte];
                op[p >> 2][p & 3] = (int)e.x;
                if ((p & 3) == 0) op[4][p >> 2] = (int)e.y;
                else op[4][p >> 2] |= (int)(e.y << (8 * (p & 3)));
            }
#pragma unroll
            for (int j = 0; j < 5; ++j)
                acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(op[j], trit_as_v4i(s.x[j]), acc[a], 0, 0, 0);
        }
    };

    Stage st[kD];
#pragma unroll
    for (int d = 0; d < kD; ++d) {
        load(st[d], d);
        // a step's loads leave before the next one's addresses are worked out (3200 -> 17280, one token: all eighteen addresses first
        // 6.85 us, so 6.65)
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                  // table ready
    int i = 0;
    for (; i + kD < items; i += kD) {
#pragma unroll
        for (int d = 0; d < kD; ++d) {
            mac(st[d], i + d);
            __builtin_amdgcn_sched_barrier(0);
            load(st[d], i + d + kD);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < kD; ++d) mac(st[d], i + d);

    if (kS > 1) {
#pragma unroll
        for (int a = 0; a < kR; ++a) fold[wave][a][lane] = acc[a];
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int a = 0; a < kR; ++a)
#pragma unroll
            for (int w = 1; w < kS; ++w) {
                const v4i o = fold[w][a][lane];
                acc[a].x += o.x; acc[a].y += o.y; acc[a].z += o.z; acc[a].w += o.w;
            }
    }
    if (r < M) {
        const float scale = yt == OutType::I32 ? 0.0f : (gamma[0] * sx[r]) / kQb;
#pragma unroll
        for (int a = 0; a < kR; ++a) {
            const int64_t n0 = (int64_t)(rb0 + a) * 16 + 4 * g;
            if (n0 < N) store_row4(y, yt, (int64_t)r * N + n0, n0, N, acc[a], scale);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// the same product with the digits left to the matrix pipe, M <= 16, x_q in LDS
// ---------------------------------------------------------------------------------------------------
// The kernel above is bound by its table: sixteen look-ups of eight bytes per 80 weights and lane, at random addresses of one 2 KB
// table, 15 clocks of the CU's LDS each (27648 x 5120 at four tokens: 11.2 us for 28 MB, here 9.4; sixteen 18.4, here
// 12.7).  What is left of the 9.4 us: the arithmetic, 74 vector instructions per lane and chunk of 5120 weights, is 5.0 of them on the
// fullest SIMDs (247 workgroups of seven row blocks, a wave each: 32 chunks where the mean is 27, at five clocks an instruction), the
// bytes 5.5, and in front of both the staging of x_q, with a quarter of a wave's weights (kD of its 16 steps) requested ahead of it.
//  Here no digit is ever formed.  With
// f_d = floor(byte / 3^d) a digit is t_d = f_d - 3 f_(d+1), so
//     sum_d x_d t_d  =  sum_(d = 0..4) x_d f_d  -  3 sum_(d = 1..4) x_(d-1) f_d,
// and the quotients are small enough for int8 operands: f_0 is the byte itself (taken as byte - 128), f_1 <= 80, f_2 <= 26, f_3 <= 8,
// f_4 <= 2, each a multiplication away for two bytes at once in the 16-bit halves of a word:
//     f_1 = (85 b + 83) >> 8,   2 f_2 = (57 b >> 8) & ~1,   2 f_3 = (19 b >> 8) & ~1,   8 f_4 = ((25 b + 46) >> 8) & ~7
// (exact for the 243 byte values; the factors are shifted out of sums of their own): 18 vector instructions for the twenty weights
// of a word.  Both sums come out of the same MFMA: eight tokens take columns 0 ... 7, and columns 8 ... 15 hold the same tokens'
// activations one digit further back.  sum_d x_d (t_d - 1) is what a row needs; the ones and the 128s are two sums over a token,
// added up once when its x_q is staged.
// x_q is staged with the columns of a quad ordered by digit, [d][p]: 16 bytes are one lane's operand of f_d.
constexpr int kTritQuadBytes = 80;
constexpr int kTritHeader = 128;                     // the tokens' corrections, 16 ints; bytes in front of a row that idle columns may read

__host__ __device__ constexpr int trit_row_bytes(int steps) { return steps * 4 * kTritQuadBytes + 16; }      // + 16: rows start on other banks

struct TritOps { v4i f[5]; };
__device__ inline uint32_t high_bytes(uint32_t even, uint32_t odd) { return __builtin_amdgcn_perm(odd, even, 0x07030501u); }
__device__ inline TritOps trit_quotients(const v4i& w) {
    TritOps o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t b = (uint32_t)w[j], e = b & 0x00FF00FFu, d = __builtin_amdgcn_perm(0u, b, 0x0c030c01u);     // bytes 0, 2 and 1, 3
        o.f[0][j] = (int)(b ^ 0x80808080u);
        o.f[1][j] = (int)high_bytes(e * 85u + 0x00530053u, d * 85u + 0x00530053u);
        o.f[2][j] = (int)(high_bytes(e * 57u, d * 57u) & 0xFEFEFEFEu);
        o.f[3][j] = (int)(high_bytes(e * 19u, d * 19u) & 0xFEFEFEFEu);
        o.f[4][j] = (int)(high_bytes(e * 25u + 0x002E002Eu, d * 25u + 0x002E002Eu) & 0xF8F8F8F8u);
    }
    return o;
}

// a row block per wave, kS waves splitting K, kW row slots (kS * kW waves), kD steps of weights in flight, kH groups of eight tokens
template <int kS, int kW, int kD, int kH>
__global__ __launch_bounds__(kS * kW * kWave) void linear_quotients_trit5(
        const int8_t* __restrict__ xq, const uint4* __restrict__ packed, const float* __restrict__ gamma, const float* __restrict__ sx,
        void* __restrict__ y, int N32, int K32, uint32_t flags /* tokens, output type */) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kThreads = kS * kW * kWave, kRsrc = 0x00020000;
    extern __shared__ uint4 smem[];
    char* const lds = reinterpret_cast<char*>(smem);
    int* const corr = reinterpret_cast<int*>(lds);
    char* const xl = lds + kTritHeader;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);          // scalar: a wave's steps, row blocks and addresses
    const int r = lane & 15, g = lane >> 4, ws = wave % kS, ww = wave / kS;
    const uint32_t K = (uint32_t)K32, N = (uint32_t)N32;
    const int M = flags_number(flags), steps = (int)((K + kTritStep - 1) / kTritStep), quads = 4 * steps;
    const uint32_t RB = (N + 15) / 16, rb = blockIdx.x * kW + ww;
    const OutType yt = flags_out_type(flags);
    const int rowbytes = trit_row_bytes(steps);

    // x_q, a quad of 80 columns per thread and round; past the row reads as zero (K is a multiple of 16)
    auto load_quad = [&](int q, v4i (&v)[5]) {
        const int m = q / quads, c = (q - m * quads) * kTritCols;
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(xq), 0, (int)(M * K), kRsrc);
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const bool in = q < M * quads && (uint32_t)(c + 16 * j) < K;
            v[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xr, in ? (int)(m * K + c + 16 * j) : -16, 0, 0));
        }
    };
    v4i xv[5];
    load_quad(tid, xv);
    if (tid < 16) corr[tid] = 0;
    __syncthreads();                                                    // (all waves' x_q loads go ahead of the weights, too)
    // the weights: a chunk per descriptor; what is not the wave's own lies past its end
    const uint64_t step_bytes = (uint64_t)RB * 1024;
    const char* wbase = reinterpret_cast<const char*>(packed) + step_bytes * (uint32_t)ws + (uint64_t)rb * 1024;
    int next = ws;
    auto load = [&](v4i& w) {
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wbase), 0, next < steps && rb < RB ? 1024 : 0, kRsrc);
        w = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, 0, 2 /* nt: read once */));
        wbase += step_bytes * kS;
        next += kS;
    };
    v4i st[kD];
#pragma unroll
    for (int d = 0; d < kD; ++d) load(st[d]);
    // the output scales of the lanes that store (token r, and r + 8)
    const float gm = gamma[0];
    float sc[kH];
#pragma unroll
    for (int h = 0; h < kH; ++h) sc[h] = yt == OutType::I32 ? 0.0f : sx[min(8 * h + (r & 7), M - 1)];
    __builtin_amdgcn_sched_barrier(0);

    for (int q = tid;;) {
        if (q < M * quads) {
            const int m = q / quads;
            char* const out = xl + m * rowbytes + (q - m * quads) * kTritQuadBytes;
            v4i o[4];
            int all = 0, first = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {                               // bytes [p][d] of 4 x 4 columns -> [d][p]
                const uint32_t a = (uint32_t)xv[j].x, b = (uint32_t)xv[j].y, c = (uint32_t)xv[j].z, d = (uint32_t)xv[j].w;
                const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u), t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
                const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u), t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
                o[0][j] = (int)__builtin_amdgcn_perm(t2, t0, 0x05040100u);
                o[1][j] = (int)__builtin_amdgcn_perm(t2, t0, 0x07060302u);
                o[2][j] = (int)__builtin_amdgcn_perm(t3, t1, 0x05040100u);
                o[3][j] = (int)__builtin_amdgcn_perm(t3, t1, 0x07060302u);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                first = __builtin_amdgcn_sdot4(o[0][j], 0x01010101, first, false);
#pragma unroll
                for (int d = 1; d < 4; ++d) all = __builtin_amdgcn_sdot4(o[d][j], 0x01010101, all, false);
                all = __builtin_amdgcn_sdot4(xv[4][j], 0x01010101, all, false);
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) *reinterpret_cast<v4i*>(out + 16 * d) = o[d];
            *reinterpret_cast<v4i*>(out + 64) = xv[4];
            int part = 127 * first - all;                               // 128 sum x_0 - sum x
            part += (int)dpp_u32<0xB1>((uint32_t)part);                 // four lanes have one step of one token
            part += (int)dpp_u32<0x4E>((uint32_t)part);
            if ((tid & 3) == 0) atomicAdd(&corr[m], part);
        }
        q += kThreads;
        if (q - tid >= M * quads) break;                                // uniform
        load_quad(q, xv);
    }
    __syncthreads();

    v4i acc[kH][4];                                                     // by quotient: f_0, f_1, f_2 and f_3, f_4
#pragma unroll
    for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[h][k] = (v4i){0, 0, 0, 0};
    const char* xr[kH];
#pragma unroll
    for (int h = 0; h < kH; ++h) xr[h] = xl + min(8 * h + (r & 7), M - 1) * rowbytes + g * kTritQuadBytes - (r & 8 ? 16 : 0);
    auto mac = [&](const v4i& w, int step) {
        if (step >= steps) return;                                      // uniform
        const int off = step * 4 * kTritQuadBytes;
        const TritOps o = trit_quotients(w);
#pragma unroll
        for (int h = 0; h < kH; ++h)
#pragma unroll
            for (int d = 0; d < 5; ++d) {
                const v4i x = *reinterpret_cast<const v4i*>(xr[h] + off + 16 * d);
                const int k = d < 3 ? d : d - 1;
                acc[h][k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(o.f[d], x, acc[h][k], 0, 0, 0);
            }
    };
    const int items = ((steps + kS - 1) / kS + kD - 1) / kD * kD;
    int i = 0;
    for (; i + kD < items; i += kD) {
#pragma unroll
        for (int d = 0; d < kD; ++d) {
            mac(st[d], ws + (i + d) * kS);
            __builtin_amdgcn_sched_barrier(0);
            load(st[d]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < kD; ++d) mac(st[d], ws + (i + d) * kS);

    // lanes r < 8 hold their token's first sum, lanes r + 8 the second
    v4i v[kH];
#pragma unroll
    for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t f = (uint32_t)acc[h][1][e] + (uint32_t)(acc[h][2][e] >> 1) + (uint32_t)(acc[h][3][e] >> 3);
            v[h][e] = (int)((uint32_t)acc[h][0][e] + f - 3u * dpp_u32<0x128>(f));              // row_ror:8; modulo 2^32, as the result fits
        }
    if (kS > 1) {
        __syncthreads();                                                // every wave is done with x_q
        v4i* const fold = reinterpret_cast<v4i*>(xl);
        if (ws > 0) {
#pragma unroll
            for (int h = 0; h < kH; ++h) fold[((ww * (kS - 1) + ws - 1) * kH + h) * kWave + lane] = v[h];
        }
        __syncthreads();
        if (ws > 0) return;
#pragma unroll
        for (int w = 0; w < kS - 1; ++w)
#pragma unroll
            for (int h = 0; h < kH; ++h) v[h] += fold[((ww * (kS - 1) + w) * kH + h) * kWave + lane];
    }
    const uint32_t n0 = rb * 16 + 4 * g;
    if (r >= 8 || n0 >= N) return;
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        const int m = 8 * h + r;
        if (m >= M) continue;
        const int c = corr[m];
        store_sums4(y, yt, (int64_t)m * N + n0, n0, N, (v4i){v[h].x + c, v[h].y + c, v[h].z + c, v[h].w + c}, (gm * sc[h]) / kQb);
    }
#endif
}

// ---------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------
hipError_t launch_unpack_trit5(const void* packed, int64_t N, int64_t K, int8_t* codes, hipStream_t stream) {
    const int64_t blocks = ceil_div(N * K, 256);
    hipLaunchKernelGGL(unpack_trit5, dim3((unsigned)(blocks < kMaxLoopBlocks ? blocks : kMaxLoopBlocks)), dim3(256), 0, stream,
                       static_cast<const uint8_t*>(packed), N, K, ceil_div(N, kRowsPerBlock), codes);
    return hipGetLastError();
}

hipError_t launch_linear_reference_trit5(const int8_t* xq, const float* sx, const void* packed, const float* gamma,
                                         int64_t M, int64_t N, int64_t K, void* y, OutType yt, hipStream_t stream) {
    const size_t ysz = yt == OutType::BF16 ? 2 : 4;
    for (int64_t m0 = 0; m0 < M; m0 += 32768) {
        const int64_t mc = (M - m0) < 32768 ? (M - m0) : 32768;
        dim3 grid((unsigned)ceil_div(N, 256), (unsigned)mc);
        hipLaunchKernelGGL(linear_reference_trit5, grid, dim3(256), 0, stream, xq + m0 * K, sx + m0,
                           static_cast<const uint8_t*>(packed), gamma, N, K, ceil_div(N, kRowsPerBlock),
                           static_cast<char*>(y) + m0 * N * ysz, yt);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------
// repacking between the two formats on the device (no weights in full precision needed)
// ---------------------------------------------------------------------------------------------------
// 320 columns are one step of the 5-trit layout (4 quads of 80) and five quads of the 2-bit layout (64 each).
//
// 5-trit -> 2-bit: a wave moves one chunk of the 5-trit layout (16 rows x 320 columns, 1 KiB in, 1280 bytes out), lane
// 16 g + r quad g of row r -- with a thread per row and step a 4096 x 11008 matrix gave the chip two wavefronts per SIMD and
// took 7.6 us (300 tokens on it, quantization and product included: 34.6 -> 33.6 us; 100 tokens on 27648 x 5120 33.4 -> 31.6).
// A 5-trit byte p of quad g holds quad columns 4p .. 4p+3, i.e. step columns 80 g + 4 p + (0 .. 3): four columns that the 2-bit
// layout keeps in one 32-bit word (word (80 g + 4 p) / 16 of the step), in field i = p & 3 of its four bytes; the table gives
// those four 2-bit codes already spread to bits 0, 8, 16, 24.  The sixteen fifth digits of a quad are step columns 80 g + 64 ..
// 80 g + 79: exactly one word.  The lane's five words go through LDS (the wave's own 1280 bytes, whose accesses complete in
// order), from where 80 lanes' worth of 16-byte quads are stored in runs of 256 bytes.
constexpr int kRepackWaves = 4;
__global__ __launch_bounds__(kRepackWaves * kWave) void repack_trit5_to_2bit(const uint4* __restrict__ in, int64_t RB, int64_t first, int64_t chunks,
                                                                             int64_t Kq2, uint4* __restrict__ out) {
    __shared__ uint2 lut[256];                       // byte -> {codes 0..3 as 2-bit fields at bits 0, 8, 16, 24; code 4}
    __shared__ __align__(16) uint32_t tiles[kRepackWaves][16 * 20];      // [row][word]; read back in 16-byte pieces
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int64_t chunk = first + (int64_t)blockIdx.x * kRepackWaves + wave;
    uint4 q = make_uint4(0, 0, 0, 0);
    if (chunk < chunks) q = in[64 * chunk + lane];
    {
        const int b = threadIdx.x;
        uint32_t sp = 0, c4 = 0;
        if (b < 243) {
#pragma unroll
            for (int d = 0; d < 4; ++d) sp |= ((uint32_t)trit5_digit(b, d) & 3u) << (8 * d);
            c4 = (uint32_t)trit5_digit(b, 4) & 3u;
        }
        lut[b] = make_uint2(sp, c4);
    }
    __syncthreads();
    if (chunk >= chunks) return;                     // whole waves; no workgroup barrier below
    const int64_t s5 = chunk / RB, rb = chunk - s5 * RB;
    uint32_t* tile = tiles[wave];
    {
        const int g = lane >> 4, r = lane & 15;
        const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
        uint32_t fifth = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint2 e = lut[(wd[j] >> (8 * i)) & 0xFFu];               // byte p = 4 j + i
                w |= e.x << (2 * i);
                fifth |= e.y << (8 * i + 2 * j);                                // column 64 + p = 64 + 4 j + i: byte i, field j
            }
            tile[r * 20 + 5 * g + j] = w;
        }
        tile[r * 20 + 5 * g + 4] = fifth;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the other lanes' words: an order for the compiler, no instruction
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = h * kWave + lane, q5 = p >> 4, r = p & 15;               // piece p: quad q5 of row r
        const int64_t kq = 5 * s5 + q5;
        if (q5 < 5 && kq < Kq2) out[quad_index_2bit(kq, rb, r, Kq2, RB)] = *reinterpret_cast<const uint4*>(tile + r * 20 + 4 * q5);
    }
}

// 2-bit -> 5-trit: the same move backwards, one thread per row and 320 columns (consecutive threads take consecutive rows of a
// 16-row block, so their 16-byte loads and stores form 256-byte runs in both layouts); 2-bit quads past the matrix's last one
// read as zero codes.
__global__ __launch_bounds__(256) void repack_2bit_to_trit5(const uint4* __restrict__ in, int64_t RB, int64_t steps5,
                                                            int64_t Kq2, uint4* __restrict__ out) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= 16 * RB * steps5) return;
    const int r = (int)(idx & 15);
    const int64_t rb = (idx >> 4) % RB, s5 = (idx >> 4) / RB;
    uint32_t words[20];
#pragma unroll
    for (int q5 = 0; q5 < 5; ++q5) {
        const int64_t kq = 5 * s5 + q5;
        uint4 q = make_uint4(0, 0, 0, 0);
        if (kq < Kq2) q = in[quad_index_2bit(kq, rb, r, Kq2, RB)];
        words[4 * q5] = q.x; words[4 * q5 + 1] = q.y; words[4 * q5 + 2] = q.z; words[4 * q5 + 3] = q.w;
    }
    // code + 1 of step column c: word c / 16, bits 8 (c & 3) + 2 ((c & 15) >> 2)
    auto digit = [&](int c) -> uint32_t {
        const uint32_t f = (words[c >> 4] >> (8 * (c & 3) + 2 * ((c & 15) >> 2))) & 3u;   // 0, 1, 3 for codes 0, +1, -1
        return f == 3u ? 0u : f + 1u;
    };
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const int c = 80 * g + 4 * p;
            const uint32_t b = digit(c) + 3 * digit(c + 1) + 9 * digit(c + 2) + 27 * digit(c + 3) + 81 * digit(80 * g + 64 + p);
            o[p >> 2] |= b << (8 * (p & 3));
        }
        out[64 * (RB * s5 + rb) + 16 * g + r] = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

hipError_t launch_repack(const void* in, bool in_trit5, int64_t N, int64_t K, void* out, hipStream_t stream) {
    const int64_t RB = ceil_div(N, kRowsPerBlock), steps5 = ceil_div(K, kTritStep), Kq2 = ceil_div(K, kColsPerQuad);
    if (!in_trit5) {
        hipLaunchKernelGGL(repack_2bit_to_trit5, dim3((unsigned)ceil_div(16 * RB * steps5, 256)), dim3(256), 0, stream, static_cast<const uint4*>(in), RB, steps5, Kq2,
                           static_cast<uint4*>(out));
        return hipGetLastError();
    }
    const int64_t chunks = RB * steps5;
    for (int64_t first = 0; first < chunks; first += kLaunchChunks) {
        const int64_t n = chunks - first < kLaunchChunks ? chunks - first : kLaunchChunks;
        hipLaunchKernelGGL(repack_trit5_to_2bit, dim3((unsigned)ceil_div(n, kRepackWaves)), dim3(kRepackWaves * kWave), 0, stream,
                           static_cast<const uint4*>(in), RB, first, first + n, Kq2, static_cast<uint4*>(out));
    }
    return hipGetLastError();
}

bool gemv_trit5_supports(int64_t M, int64_t N, int64_t K, const void* xq) {
    // the launch of a matrix tall enough to pass a grid: 128 threads for two row blocks
    return M >= 1 && M <= 16 && K % 16 == 0 && reinterpret_cast<uintptr_t>(xq) % 16 == 0 && ceil_div(N, 2 * kRowsPerBlock) * 128 < kMaxGridThreads;
}

template <int kR, int kS, int kD>
static void launch_trit5(const int8_t* xq, const float* sx, const void* packed, const float* gamma, int64_t M, int64_t N,
                         int64_t K, void* y, OutType yt, hipStream_t stream, LaunchPlan* plan) {
    const int RB = (int)ceil_div(N, kRowsPerBlock);
    if (plan) return plan->set("trit5_decode", {kR, kS, kD}, (unsigned)ceil_div(RB, kR), 1, kS * kWave, 0, 1);
    hipLaunchKernelGGL((linear_gemv16_trit5<kR, kS, kD>), dim3((unsigned)ceil_div(RB, kR)), dim3(kS * kWave), 0, stream, xq,
                       static_cast<const uint4*>(packed), gamma, sx, y, (int)N, (int)K, product_flags(0, yt) | (uint32_t)M << 4);
}

// Where the quotients are the faster form, and in which launch shape (six choices over 22 widths of 200 ... 5000 row blocks, 1 ... 30
// steps, eight token counts; us, table / quotients).  What decides:
//   * the table's time grows with every token, the quotients' with every group of eight: 8 or 16 tokens go to the quotients earlier
//     than 5 or 9 do (16480 x 2496, nine tokens 6.2 / 7.6, sixteen 7.5 / 7.7; 40000 x 7616 21.3 / 25.4, 29.0 / 31.0);
//   * staging x_q and its sums come in front of the first product, so short walks on few row blocks stay with the table (4320 x 2496,
//     nine tokens 4.0 / 4.7; 8320 x 2496, five 4.3 / 5.1), and long ones leave it (600 x 8000, one token 4.7 / 4.4; 16384 x 8000, four
//     13.1 / 9.6, sixteen 22.1 / 13.2; 57344 x 8192, sixteen 47.8 / 34.9);
//   * a launch takes as long as its fullest CU: eight row blocks per workgroup up to 2048, where that is one workgroup each, and from
//     3072; in between the table's workgroups are dealt out more evenly, and with few tokens in the last group it wins (32960 x 9536,
//     nine tokens 24.7 / 34.3), else four row blocks with K split in two take half the step from one round to the next;
//     one workgroup on every CU where eight, six or five row blocks are too many or too few for that: five or six with K split in two from
//     ten steps on (eight tokens: 20480 x 8192 14.9 / 12.0, 17280 x 3200 7.3 / 6.8; sixteen, 22016 x 4096 11.4 / 10.0; with few tokens four
//     waves a row block hide more: three 21424 x 4608 9.4 / 8.8, 24560 x 3968 8.8 / 8.4, four 20496 x 3520 7.5 / 7.1;
//     five on up to 1280 row blocks from thirteen steps on), seven and eight without a split for up to four (27648 x 5120 10.2 / 9.7, 32640 x 8320 13.0 / 12.6);
//   * the table walks whole rounds of four steps on wide layers: there its best counts are four and eight.
// The picks are within 5 % of the faster of table and previous picks wherever measured.  x_q has to fit the LDS.
struct QuotientForm { int s, w, d; };                  // kS, kW, kD; none: s = 0
static QuotientForm pick_quotients(int64_t M, int64_t RB, int64_t steps) {
    constexpr QuotientForm table{0, 0, 0}, eight{1, 8, 4}, seven{1, 7, 4}, six{2, 6, 2}, five{2, 5, 2}, four{2, 4, 2}, two{4, 2, 2}, one{4, 1, 2}, one_long{8, 1, 2};
    if (RB <= 256) return M <= 8 && steps >= 20 && (M <= 4 || M > 6 || steps < 28) ? one_long : table;
    if (RB <= 512) {
        if (M <= 4) return steps >= 20 ? one_long : table;
        return steps >= (M > 12 || (M > 6 && M <= 8) ? 10 : 14) ? two : table;
    }
    if (RB <= 1024) {
        const bool narrow = RB <= 768, middle = steps >= 6 && steps <= 8;
        if (M <= 4) {
            if (steps <= 4) return narrow ? one : four;
            if (steps < 10) return table;
            return M == 1 || steps < 20 ? one : two;
        }
        if (M <= 8) {
            if (narrow && steps <= 5) return one;
            if (narrow && M <= 6) return steps < 14 ? table : one_long;
            return middle && (narrow || M <= 6) ? table : four;
        }
        if (M <= 10) return (narrow ? steps >= 4 && steps < 14 : middle) ? table : four;
        return narrow && middle && M <= 12 ? table : four;
    }
    if (RB <= 1536 && steps >= (M == 5 && RB <= 1280 ? 13 : 10) && (M > 4 || (M == 4 && RB > 1360))) return RB <= 1280 ? five : six;
    if (M <= 4 && RB > 1536 && RB <= 2048) return RB <= 1792 ? seven : eight;
    if (M <= 4) {
        if (RB >= 3072) return eight;
        if (RB > 2048 && steps == 4) return table;
        if (RB >= 1536) return four;
        if (steps <= 4) return four;
        return M == 1 || steps < 20 ? one : two;
    }
    if (RB < 1536) {
        if (M <= 8) return steps <= 3 ? eight : M <= 6 || steps <= 8 ? one : two;             // fewer than ten steps, or thirteen
        if (M <= 10 && steps >= 5 && (RB <= 1280 || steps <= 8)) return table;
        return M <= 12 && steps >= 6 && steps <= 8 ? table : eight;
    }
    if (RB > 2048 && RB < 3072) {
        if (steps <= 2) return eight;
        if (steps == 4) return table;
        if (M <= 8) return four;
        if (M <= 12 && (RB <= 2816 || steps == 3)) return table;
        if (steps <= 5) return eight;
        if (M <= 10 && steps == 8) return table;
        return M > 12 && RB <= 2816 && (steps == 8 || steps >= 16) ? table : four;
    }
    if (steps == 8 && (M == 9 || M == 10)) return table;
    return steps == 4 && RB > 2048 && M > 8 && (M <= 12 || RB < 3600) ? table : eight;
}
constexpr int64_t kTritMaxLds = 160 * 1024;

template <int kS, int kW, int kD>
static bool launch_quotients(const int8_t* xq, const float* sx, const void* packed, const float* gamma, int64_t M, int64_t N,
                             int64_t K, void* y, OutType yt, hipStream_t stream, LaunchPlan* plan, hipError_t* status) {
    if (M > 8 && (kW == 1 || kW == 7)) return false;       // not picked for two groups of eight tokens, and not built
    const int64_t rows = M * trit_row_bytes((int)ceil_div(K, kTritStep)), fold = (int64_t)(kS - 1) * kW * (M <= 8 ? 1 : 2) * 1024;
    const int64_t lds = kTritHeader + (rows > fold ? rows : fold), wgs = ceil_div(ceil_div(N, kRowsPerBlock), kW);
    if (lds > kTritMaxLds || wgs * kS * kW * kWave >= kMaxGridThreads) return false;
    if (plan) {
        plan->set("trit5_decode", {kS, kW, kD, M <= 8 ? 1 : 2}, (unsigned)wgs, 1, kS * kW * kWave, (size_t)lds, 1);
        return true;
    }
    auto go = [&](auto* kernel, RaisedFlags& raised) -> hipError_t {
        if (lds > 65536) {
            const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)kTritMaxLds, raised);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(kS * kW * kWave), lds, stream, xq, static_cast<const uint4*>(packed), gamma, sx, y,
                           (int)N, (int)K, product_flags(0, yt) | (uint32_t)M << 4);
        return hipGetLastError();
    };
    static RaisedFlags one = {}, two = {};
    if (M <= 8) {
        *status = go(linear_quotients_trit5<kS, kW, kD, 1>, one);
    } else if constexpr (kW != 1 && kW != 7) {
        *status = go(linear_quotients_trit5<kS, kW, kD, 2>, two);
    }
    return true;
}

hipError_t launch_linear_gemv_trit5(const int8_t* xq, const float* sx, const void* packed, const float* gamma,
                                    int64_t M, int64_t N, int64_t K, void* y, OutType yt, hipStream_t stream, LaunchPlan* plan) {
    const int64_t RB = ceil_div(N, kRowsPerBlock);
    const int64_t steps = ceil_div(K, kTritStep);
    const QuotientForm f = pick_quotients(M, RB, steps);
    hipError_t e = hipSuccess;
#define FORM(S_, W_, D_) if (f.s == S_ && f.w == W_ && f.d == D_ && launch_quotients<S_, W_, D_>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan, &e)) return e
    FORM(8, 1, 2);
    FORM(4, 1, 2);
    FORM(4, 2, 2);
    FORM(2, 4, 2);
    FORM(2, 5, 2);
    FORM(2, 6, 2);
    FORM(1, 7, 4);
    FORM(1, 8, 4);
#undef FORM
    // the share of a wave's padded K walk (a multiple of the prefetch depth) that is real steps
    auto walk = [&](int ks, int kd) { return (double)steps / (double)(ceil_div(ceil_div(steps, (int64_t)ks), (int64_t)kd) * kd * ks); };
    // Measured on MI355X, M = 1, fifteen forms per shape: 3200 -> 3200 4.0 -> 3.5 us and 3200 -> 17280 8.0 -> 6.6 us with
    // depth 3 (ten steps fill three rounds of four waves exactly; thirteen steps would walk 24), 4096 -> 22016 9.4 -> 8.7 us
    // and 28672 -> 8192 17.9 -> 15.5 us with two row blocks per wave.
    if (RB >= 2048)                                   launch_trit5<2, 2, 2>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    else if (steps >= 64 && RB >= 512)                launch_trit5<2, 8, 2>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    else if (steps >= 24)                             launch_trit5<1, 8, 2>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    else if (walk(4, 3) > walk(4, 2))                 launch_trit5<1, 4, 3>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    else if (RB >= 1024)                              launch_trit5<2, 4, 2>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    else                                              launch_trit5<1, 4, 2>(xq, sx, packed, gamma, M, N, K, y, yt, stream, plan);
    return plan ? hipSuccess : hipGetLastError();
}

}  // namespace bitnet
