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

// One store of sizeof(V) bytes at any alignment: the hardware takes it, and splits it where it crosses a line.
template <typename V> __device__ inline void store_any(void* p, const V& v) { __builtin_memcpy(p, &v, sizeof(V)); }

__device__ inline uint2 bf16x4(const v4i& v, float scale) {
    const uint32_t a = f32_to_bf16((float)v.x * scale), b = f32_to_bf16((float)v.y * scale);
    const uint32_t c = f32_to_bf16((float)v.z * scale), d = f32_to_bf16((float)v.w * scale);
    return make_uint2(a | b << 16, c | d << 16);
}

// Four consecutive outputs of a token, the integer sums v, from row n0 on: one store, also where N is no multiple of four or the
// base is aligned to no more than an output; by the element only across a row's end.  (By the element wherever N or the base were not
// aligned, us / this: 64 tokens, 4096 -> 9999 9.0 / 8.25, 12 tokens, 4096 -> 4095 3.4 / 3.07.)
__device__ inline void store_sums4(void* y, OutType yt, int64_t base, int64_t n0, int64_t N, const v4i& v, float scale) {
    if (__builtin_expect(n0 + 4 <= N, 1)) {
        if (yt == OutType::BF16) store_any(static_cast<uint16_t*>(y) + base, bf16x4(v, scale));
        else if (yt == OutType::F32)
            store_any(static_cast<float*>(y) + base, make_float4((float)v.x * scale, (float)v.y * scale, (float)v.z * scale, (float)v.w * scale));
        else store_any(static_cast<int32_t*>(y) + base, v);
        return;
    }
    const int s[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (n0 + e >= N) continue;
        if (yt == OutType::BF16) static_cast<uint16_t*>(y)[base + e] = f32_to_bf16((float)s[e] * scale);
        else if (yt == OutType::F32) static_cast<float*>(y)[base + e] = (float)s[e] * scale;
        else static_cast<int32_t*>(y)[base + e] = s[e];
    }
}
// ... which still carry the decode factor 64 (dropped exactly)
__device__ inline void store_row4(void* y, OutType yt, int64_t base, int64_t n0, int64_t N, const v4i& s, float scale) {
    store_sums4(y, yt, base, n0, N, (v4i){s.x >> 6, s.y >> 6, s.z >> 6, s.w >> 6}, scale);
}

// Waits until at most kN vector-memory loads are in flight: the oldest have arrived.
template <int kN>
__device__ inline void wait_loads() {                  // imm: vmcnt[3:0] | expcnt 7 << 4 | lgkmcnt 15 << 8 | vmcnt[5:4] << 14
    __builtin_amdgcn_s_waitcnt((kN & 15) | 0x0F70 | ((kN >> 4) << 14));
}
// The outputs of a wave's kR row blocks and kMT token tiles: four consecutive ones of a token per lane, in one store.  As four stores of
// two bytes, each behind its own choice of the type, they were most of the 1.2 us between a 29-token launch's last product and its
// end.  Only a wave with a row block that N cuts short looks at each lane's rows: with that test, and the stores by the element behind it, in
// front of every store, launches of a short K took 0.2 us more (117 tokens, 96 -> 11136 5.39 / 5.71).
template <int kMT, int kR>
__device__ inline void store_tiles(void* y, OutType yt, int64_t N, int M, int rbw, const v4i (&acc)[kR][kMT], const float (&gm)[kR],
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
                const v4i v = {acc[a][t].x >> 6, acc[a][t].y >> 6, acc[a][t].z >> 6, acc[a][t].w >> 6};       // drops the decode factor 64, exactly
                put((int64_t)m * N + n0, n0, v, (gm[a] * sxm[t]) / kQb);
            }
        }
    };
    if (__builtin_expect((int64_t)(rbw + kR) * 16 > N, 0))
        each([&](int64_t at, int64_t n0, const v4i& v, float scale) { if (n0 < N) store_sums4(y, yt, at, n0, N, v, scale); });
    else if (yt == OutType::BF16) each([&](int64_t at, int64_t, const v4i& v, float scale) { store_any(static_cast<uint16_t*>(y) + at, bf16x4(v, scale)); });
    else if (yt == OutType::F32)
        each([&](int64_t at, int64_t, const v4i& v, float scale) {
            store_any(static_cast<float*>(y) + at, make_float4((float)v.x * scale, (float)v.y * scale, (float)v.z * scale, (float)v.w * scale));
        });
    else each([&](int64_t at, int64_t, const v4i& v, float) { store_any(static_cast<int32_t*>(y) + at, v); });
}

}  // namespace bitnet
