// Batched decode with the K steps dealt out to the waves of a workgroup: the weight-streaming product of linear_skinny.hip (same
// packed layout, decode and v_mfma_i32_16x16x64_i8 contraction, same results bit for bit) for its smaller workgroup tiles.
#include "gemv_common.hpp"

namespace bitnet {

// s_waitcnt where nothing was requested behind a tile but the copies of `tiles` more (a constant once the loop is unrolled)
__device__ inline void wait_loads_last(int tiles) {
    switch (tiles) {
        case 0: wait_loads<0>(); break;
        case 1: wait_loads<4>(); break;
        case 2: wait_loads<8>(); break;
        case 3: wait_loads<12>(); break;
        default: wait_loads<16>(); break;
    }
}

// A workgroup owns kR * kW row blocks and 16 kMT tokens, and each of its kS * kW waves all of them for every (kS kW)-th K step.  What
// a wave multiplies nobody else reads, so that nothing in the K loop is shared: a wave copies its activations to LDS slots of its
// own, waits for them by its own count of loads in flight, and meets the others once, where the partial sums are folded.
// The kernels of linear_skinny.hip, whose waves share the activations of a step, meet at a barrier per step; at 29 tokens on
// 4096 columns, four steps a wave, that chain of barriers was most of the launch.
//
// What bounds it.  A launch that does nothing takes 2.1 us in a graph.  29 tokens, 4096 -> 12288: weights at the rate of HBM 2.4 us,
// x_q out of the L2s 1.0 (every workgroup pulls all of its tokens: 30 MB), fold and store 1.6, hidden in part: 6.7.  300 tokens, 11008
// -> 4096: 250 MB through the L2s 7 us, 27 GOP 7, LDS (each byte of x_q written once and read once) 6, overlapped by the ring:
// a wave's slots hold a tile of 16 tokens and 256 columns each, and a slot is requested again, one step on, as soon as its tile
// has been multiplied, so that the others' loads are under way meanwhile.  With a step as the unit (requested, waited for and
// multiplied as a whole) the same launch took 18.5 us instead of 17.9, 128 tokens 10.9 instead of 10.2, 29 on 4096 -> 12288 6.5 / 6.3.
// A second step's slots in LDS made every form 2-8 % slower (29 tokens 4096 -> 4096 3.61 / 3.93: more code in front of a launch of
// two steps a wave), half a step's 2-5 % (128 tokens 11008 -> 4096 10.0 / 10.3; one form has them), sixteen waves instead of eight all but
// the longest K.
//
// us in a graph, weights from HBM, linear_skinny.hip / this: 16 tokens 4096 -> 4096 3.56 / 3.24, 11008 -> 4096 6.46 / 5.83; 29 tokens
// 4096 -> 4096 4.21 / 3.56, -> 12288 6.83 / 6.68, -> 22016 8.70 / 8.48, 11008 -> 4096 7.26 / 6.38; 64 tokens 4.62 / 4.28 and 9.09 /
// 8.05; 128 tokens 6.11 / 5.6 and 12.74 / 10.3; 200 tokens 8.71 / 7.87 and 17.9 / 13.9; 300 tokens 11008 -> 4096 22.4 / 17.9.  Over 300
// random sizes of 5 ... 512 tokens, 256 ... 16384 rows and 256 ... 11200 columns, geometric mean 1.18.
// Accumulators, decoded weights and the next step's take 20 kRows + 4 kRows kMT registers: eight row blocks of 32 tokens or six of 64 spill.
template <int kMT, int kR, int kW, int kS, int kQ>
__global__ __launch_bounds__(kS * kW * kWave) void linear_ksplit_2bit(
        // 14 dwords (product_flags says why); blockIdx.z selects a tile of 16 * kMT tokens
        const int8_t* __restrict__ xq_all, const uint4* __restrict__ packed, const float* __restrict__ gamma,
        const float* __restrict__ sx_all, void* __restrict__ yv, int N32, int K32, uint32_t flags /* tokens, output type, gamma stride */) {
#if defined(__HIP_DEVICE_COMPILE__)      // the buffer-resource builtins exist in the device pass only
    extern __shared__ uint4 smem[];
    constexpr int kRows = kR * kW, kWaves = kS * kW, kTiles = kRows * kMT, kSlot = 16 * 256;
    const int64_t K = K32, N = N32;
    const int Kq = (K32 + kColsPerQuad - 1) / kColsPerQuad;
    const int RB = (int)((N + kRowsPerBlock - 1) / kRowsPerBlock), M_all = flags_number(flags), gstride = flags_gstride(flags);
    const OutType yt = flags_out_type(flags);
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int steps = (Kq + 3) >> 2, tail_quads = 16 * (Kq - 4 * (steps - 1));
    const int m0 = blockIdx.z * (16 * kMT), M = min(M_all - m0, 16 * kMT), rb0 = blockIdx.x * kRows;
    const int n = (steps - wave + kWaves - 1) / kWaves;                // steps of this wave: wave + i * kWaves; none where it is <= 0
    char* slots = reinterpret_cast<char*>(smem) + wave * (kQ * kSlot);

    // Activation copies: lane i of copy c of a tile fills chunk slot i & 15 of token 4 c + (i >> 4) with chunk (i & 15) ^ token.  The
    // whole byte offset travels in the vector offset, which the hardware range check covers: past the last token zeros arrive.
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t*>(xq_all + (int64_t)m0 * K), 0, (int)min((int64_t)M * K, (int64_t)0x7FFFFFFF), 0x00020000);
    uint32_t xoff[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int row = 4 * c + (lane >> 4);
        xoff[c] = (uint32_t)row * (uint32_t)K32 + (uint32_t)(((lane & 15) ^ row) << 4) + (uint32_t)wave * 256u;
    }
    auto copy_x = [&](int i, int t, int slot) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, (__attribute__((address_space(3))) void*)(slots + (4 * slot + c) * 1024), 16,
                                                     xoff[c] + (uint32_t)(i * (kWaves * 256) + t * 16 * K32), 0, 0, 0);
    };
    // Weight quads: one K step of the packed layout as a raw buffer; a row block's chunk is 64 quads in a whole step, tail_quads in a
    // partial last one, where lanes past it are clamped here and masked in decode().
    auto load_w = [&](uint4 (&w)[kRows], int i) {
        const int sl = wave + i * kWaves, quads = sl == steps - 1 ? tail_quads : 64;
        const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(packed + (int64_t)sl * RB * 64), 0, RB * 1024, 0x00020000);
        const int at = min(lane, quads - 1) * 16;
#pragma unroll
        for (int a = 0; a < kRows; ++a)
            w[a] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, at, min(rb0 + a, RB - 1) * quads * 16, 0));
    };

    v4i acc[kRows][kMT];
#pragma unroll
    for (int a = 0; a < kRows; ++a)
#pragma unroll
        for (int t = 0; t < kMT; ++t) acc[a][t] = (v4i){0, 0, 0, 0};
    uint4 w[kRows];
    v4i A[4][kRows];
    auto decode = [&](int i) {
        const uint32_t km = lane < (wave + i * kWaves == steps - 1 ? tail_quads : 64) ? 0xC0C0C0C0u : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int a = 0; a < kRows; ++a) A[j][a] = decode_word_masked(quad_word(w[a], j), km);
    };
    auto multiply = [&](int t, int slot) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const v4i X = *reinterpret_cast<const v4i*>(slots + slot * kSlot + r * 256 + (((4 * g + j) ^ r) << 4));
#pragma unroll
            for (int a = 0; a < kRows; ++a) acc[a][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[j][a], X, acc[a][t], 0, 0, 0);
        }
    };

    // Loads are counted in issue order: the weights of a step before the copies of its tiles, tile by tile.  The fences pin that order,
    // and the build reads it off the assembly.
    if (n > 0) {
        load_w(w, 0);
        issue_fence();
#pragma unroll
        for (int u = 0; u < kQ; ++u)
            if (u < kMT || n > u / kMT) {
                copy_x(u / kMT, u % kMT, u);
                issue_fence();
            }
    }
    // The output scales of the tiles that this wave will fold, tile q kWaves + wave (row block tile / kMT, token tile tile % kMT).
    constexpr int kMine = (kTiles + kWaves - 1) / kWaves;
    float gm[kMine][1], sxm[kMine][1];
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const int tile = min(q * kWaves + wave, kTiles - 1), a = tile / kMT, t = tile - a * kMT;
        gm[q][0] = gamma[gstride * min(rb0 + a, RB - 1)];
        sxm[q][0] = yt == OutType::I32 ? 0.0f : sx_all[m0 + min(16 * t + r, M - 1)];
    }
    issue_fence();
    // Tile u = i kMT + t lies in slot u % kQ; behind it that slot is requested for tile u + kQ.  Younger than its own copies, at
    // its turn, are those of the kQ - 1 tiles that follow it and at least the weights of the next step.
    constexpr int kAhead = (kQ + kMT - 1) / kMT;       // steps that the slots reach ahead, the last one perhaps in part
    int i = 0, slot = 0;
    for (; i + kAhead < n; ++i) {
        decode(i);
        load_w(w, i + 1);
        issue_fence();
#pragma unroll
        for (int t = 0; t < kMT; ++t) {
            const int at = kQ == kMT ? t : slot;
            wait_loads<4 * (kQ - 1) + kRows>();
            issue_fence();
            multiply(t, at);
            issue_fence();
            __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): the tile has been read, its slot is free
            copy_x(i + (t + kQ) / kMT, (t + kQ) % kMT, at);
            issue_fence();
            slot = slot + 1 == kQ ? 0 : slot + 1;
        }
    }
    // the last kAhead steps, of which a wave with fewer has none: what is not there is not requested
#pragma unroll
    for (int e = kAhead - 1; e >= 0; --e) {
        if (n <= e) continue;
        i = n - 1 - e;
        decode(i);
        if (e > 0) load_w(w, i + 1);
        issue_fence();
#pragma unroll
        for (int t = 0; t < kMT; ++t) {
            const int left = e * kMT + kMT - 1 - t;                    // tiles behind this one
            const int at = kQ == kMT ? t : slot;
            wait_loads_last(left < kQ - 1 ? left : kQ - 1);
            issue_fence();
            multiply(t, at);
            issue_fence();
            if (left >= kQ) {
                __builtin_amdgcn_s_waitcnt(0xC07F);
                copy_x(i + (t + kQ) / kMT, (t + kQ) % kMT, at);
                issue_fence();
            }
            slot = slot + 1 == kQ ? 0 : slot + 1;
        }
    }

    // Fold: every wave's partial tiles through LDS, where the slots were; a wave adds up and stores the tiles that are its own.  Where
    // the slots do not hold all partials (32 tokens by six row blocks: 96 KiB over 64) the upper half of the waves hands its own to the lower half
    // first.
    constexpr bool kHalves = kWaves * kTiles * 1024 > kWaves * kQ * kSlot;
    constexpr int kTop = kHalves ? kWaves / 2 : kWaves;
    static_assert(kTop * kTiles * 1024 <= kWaves * kQ * kSlot, "the fold reuses the activation slots");
    v4i* fold = reinterpret_cast<v4i*>(smem);
    __syncthreads();
    auto park = [&](int at) {
#pragma unroll
        for (int a = 0; a < kRows; ++a)
#pragma unroll
            for (int t = 0; t < kMT; ++t) fold[(at * kTiles + a * kMT + t) * kWave + lane] = acc[a][t];
    };
    if constexpr (kHalves) {
        if (wave >= kTop) park(wave - kTop);
        __syncthreads();
        if (wave < kTop) {
#pragma unroll
            for (int a = 0; a < kRows; ++a)
#pragma unroll
                for (int t = 0; t < kMT; ++t) acc[a][t] += fold[(wave * kTiles + a * kMT + t) * kWave + lane];
            park(wave);                                // over what this wave alone has read
        }
    } else {
        park(wave);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const int tile = q * kWaves + wave, a = tile / kMT, t = tile - a * kMT;
        if (tile >= kTiles) break;
        v4i sum[1][1] = {{fold[tile * kWave + lane]}};
#pragma unroll
        for (int u = 1; u < kTop; ++u) sum[0][0] += fold[(u * kTiles + tile) * kWave + lane];
        void* y = static_cast<char*>(yv) + (int64_t)(m0 + 16 * t) * N * (yt == OutType::BF16 ? 2 : 4);
        store_tiles<1, 1>(y, yt, N, M - 16 * t, rb0 + a, sum, gm[q], sxm[q]);
    }
#endif
}

// kLx + 1 stages of 16 kMT tokens per group of kW waves, shared out to them as slots of 16 tokens
template <int kMT, int kR, int kW, int kS, int kLx>
static hipError_t launch(const int8_t* xq, const float* sx, const void* packed, const float* gamma, int gstride, int64_t M, int64_t N, int64_t K,
                         void* y, OutType yt, hipStream_t stream, LaunchPlan* plan) {
    constexpr int kQ = (kLx + 1) * kMT / kW;
    static_assert(kQ >= kMT && kQ * kW == (kLx + 1) * kMT, "a whole step of slots for each wave");
    constexpr size_t lds = (size_t)kS * kW * kQ * 4096;
    static_assert(lds <= 160 * 1024 && kS * kW <= 16, "a CU's LDS, 1024 threads");
    auto* kern = linear_ksplit_2bit<kMT, kR, kW, kS, kQ>;
    const dim3 grid((unsigned)ceil_div(ceil_div(N, kRowsPerBlock), kR * kW), 1, (unsigned)ceil_div(M, 16 * kMT));
    if (plan) {
        plan->set("batched_decode", {kMT, kR, kW, kS, 2, kLx}, grid.x * grid.z, 1, kS * kW * kWave, lds, 1);
        return hipSuccess;
    }
    if (lds > 65536) {
        static RaisedFlags raised = {};
        const hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, grid, dim3(kS * kW * kWave), lds, stream, xq, static_cast<const uint4*>(packed), gamma, sx, y, (int)N, (int)K,
                       product_flags(gstride, yt) | (uint32_t)M << 4);
    return hipGetLastError();
}

bool launch_linear_ksplit_2bit(int kmt, int rows, const int8_t* xq, const float* sx, const void* packed, const float* gamma, int gstride, int64_t M,
                               int64_t N, int64_t K, void* y, OutType yt, hipStream_t stream, LaunchPlan* plan, hipError_t* status) {
#define KSPLIT(MT_, R_, W_, S_, LX_) \
    if (kmt == MT_ && rows == R_ * W_) { \
        *status = launch<MT_, R_, W_, S_, LX_>(xq, sx, packed, gamma, gstride, M, N, K, y, yt, stream, plan); \
        return true; \
    }
    KSPLIT(1, 1, 1, 8, 0)
    KSPLIT(1, 1, 2, 4, 1)
    KSPLIT(1, 2, 2, 4, 1)
    KSPLIT(2, 1, 1, 8, 0)
    KSPLIT(2, 1, 2, 4, 1)
    KSPLIT(2, 2, 2, 4, 2)
    KSPLIT(2, 6, 1, 8, 0)
    KSPLIT(4, 1, 1, 8, 0)
    KSPLIT(4, 4, 1, 8, 0)
    KSPLIT(5, 4, 1, 8, 0)
#undef KSPLIT
    return false;
}
}  // namespace bitnet
