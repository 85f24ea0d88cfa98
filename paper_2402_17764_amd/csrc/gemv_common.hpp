// Pieces shared by the weight-streaming BitLinear kernels (decode, M <= 16, and batched decode, M <= 64).
#pragma once
#include "bitnet_device.hpp"
#include "bitnet_internal.hpp"

namespace bitnet {

typedef int v4i __attribute__((ext_vector_type(4)));

// One packed word (16 codes) -> the four int8 operand registers of an MFMA, 64 * code in every byte:
// (w << (6 - 2 i)) & 0xC0C0C0C0 for register i.  The lane's validity is folded into the constant: km is
// 0xC0C0C0C0, or 0 for lanes and steps whose weights must not count.
__device__ inline v4i decode_word_masked(uint32_t w, uint32_t km) {
    v4i a;
    a.x = (int)((w << 6) & km);
    a.y = (int)((w << 4) & km);
    a.z = (int)((w << 2) & km);
    a.w = (int)(w & km);
    return a;
}

__device__ inline v4i as_v4i(const uint4& u) {
    v4i a;
    a.x = (int)u.x; a.y = (int)u.y; a.z = (int)u.z; a.w = (int)u.w;
    return a;
}

__device__ inline uint32_t quad_word(const uint4& q, int j) { return j == 0 ? q.x : j == 1 ? q.y : j == 2 ? q.z : q.w; }

// Pins the order of memory instructions for kernels that count loads in flight: nothing moves across
// it, neither in the optimizer nor in the instruction scheduler.
__device__ inline void issue_fence() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

__device__ inline void store_row4(void* y, OutType yt, int64_t base, int64_t n0, int64_t N, const v4i& s, float scale) {
    const int v[4] = {s.x >> 6, s.y >> 6, s.z >> 6, s.w >> 6};   // drop the decode factor 64 (exact)
    if (yt == OutType::I32) {
        int32_t* yo = static_cast<int32_t*>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n0 + e < N) yo[base + e] = v[e];
    } else if (yt == OutType::F32) {
        float* yo = static_cast<float*>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n0 + e < N) yo[base + e] = (float)v[e] * scale;
    } else {
        uint16_t* yo = static_cast<uint16_t*>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n0 + e < N) yo[base + e] = f32_to_bf16((float)v[e] * scale);
    }
}

// Waits until at most kN vector-memory loads are in flight: the oldest have arrived.
template <int kN>
__device__ inline void wait_loads() {                  // imm: vmcnt[3:0] | expcnt 7 << 4 | lgkmcnt 15 << 8 | vmcnt[5:4] << 14
    __builtin_amdgcn_s_waitcnt((kN & 15) | 0x0F70 | ((kN >> 4) << 14));
}
// The outputs of a wave's kR row blocks and kMT token tiles: four consecutive ones of a token per lane, in one store where rows and
// base allow it (flags_vec_store; N is then a multiple of four).  As four stores of two bytes, each behind its own choice of the
// type, they were most of the 1.2 us between a 29-token launch's last product and its end.
template <int kMT, int kR>
__device__ inline void store_tiles(void* y, OutType yt, bool wide, int64_t N, int M, int rbw, const v4i (&acc)[kR][kMT], const float (&gm)[kR],
                                   const float (&sxm)[kMT]) {
    const int lane = threadIdx.x & (kWave - 1), r = lane & 15, g = lane >> 4;
    auto each = [&](auto&& put) {
#pragma unroll
        for (int t = 0; t < kMT; ++t) {
            const int m = 16 * t + r;                                  // MFMA output column = token
            if (m >= M) continue;
#pragma unroll
            for (int a = 0; a < kR; ++a) {
                const int64_t n0 = (int64_t)(rbw + a) * 16 + 4 * g;
                if (n0 < N) put((int64_t)m * N + n0, n0, acc[a][t], (gm[a] * sxm[t]) / kQb);
            }
        }
    };
    // (>> 6 drops the decode factor 64, exactly)
    if (!wide) each([&](int64_t at, int64_t n0, const v4i& v, float scale) { store_row4(y, yt, at, n0, N, v, scale); });
    else if (yt == OutType::BF16)
        each([&](int64_t at, int64_t, const v4i& v, float scale) {
            const uint32_t a = f32_to_bf16((float)(v.x >> 6) * scale), b = f32_to_bf16((float)(v.y >> 6) * scale);
            const uint32_t c = f32_to_bf16((float)(v.z >> 6) * scale), d = f32_to_bf16((float)(v.w >> 6) * scale);
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(y) + at) = make_uint2(a | b << 16, c | d << 16);
        });
    else if (yt == OutType::F32)
        each([&](int64_t at, int64_t, const v4i& v, float scale) {
            *reinterpret_cast<float4*>(static_cast<float*>(y) + at) =
                make_float4((float)(v.x >> 6) * scale, (float)(v.y >> 6) * scale, (float)(v.z >> 6) * scale, (float)(v.w >> 6) * scale);
        });
    else
        each([&](int64_t at, int64_t, const v4i& v, float) {
            *reinterpret_cast<int4*>(static_cast<int32_t*>(y) + at) = make_int4(v.x >> 6, v.y >> 6, v.z >> 6, v.w >> 6);
        });
}

// four consecutive outputs from a multiple of four on are one aligned store
inline bool wide_rows(const void* y, int64_t N, OutType yt) {
    return N % 4 == 0 && reinterpret_cast<uintptr_t>(y) % (yt == OutType::BF16 ? 8 : 16) == 0;
}

}  // namespace bitnet
