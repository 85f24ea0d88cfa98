// Absmean ternary weight quantization (Eq. (1)-(3) of arXiv 2402.17764) for gfx950.
//
//   pass 1  abs_sum_partials : grid-stride |W| sum, double-double per thread, fixed-shape tree
//                              inside the block, one (hi, lo) pair per block into the workspace
//   pass 2                   : gamma = fp32(S / (N K)); done at the top of pass 3 (one launch and 4.5 us less)
//   pass 3  ternarize_pack   : re-reads W from its end (what pass 1 read last is still in the memory-side
//                              cache), takes the decision of Eq. (1)-(2) in fp32 and writes the packed
//                              layout one 1 KiB (row block, K step) chunk per workgroup pass
//
// From 96 MiB of W on (128 of bf16, more for narrow matrices; and a workspace with room for it) the two reads become one: a sample of W bounds gamma, and with it
// the threshold of Eq. (1)-(2), so that one pass adds up |W| and codes every weight but the few between the bounds
// (guess_pack_2bit below).
//
// Otherwise the path is HBM-bound at 8.25 B per fp32 weight, 4.25 per bf16 one (two reads of W, one packed write).  Both reading passes
// are shaped by what a plain read loop reaches on this chip: 8 waves per CU with four 16-byte loads each in
// flight read 6.1-6.2 TB/s, 32 waves per CU 5.1-5.3 TB/s.
#include "bitnet_device.hpp"
#include "bitnet_internal.hpp"

namespace bitnet {

// ---------------------------------------------------------------------------------------------------
// pass 1
// ---------------------------------------------------------------------------------------------------
constexpr int kSumThreads = 512;
constexpr int kSumBlocks = 256;                           // one per CU: 8 waves per CU
constexpr int kSumLoads = 4;                              // 16-byte loads in flight per thread

__device__ inline float widen1(float v) { return v; }
__device__ inline float widen1(uint16_t v) { return bf16_to_f32(v); }

// |.| of the 4 (fp32) or 8 (bf16) elements of one 16-byte vector, added to the accumulators.
//
// bf16: eight magnitudes of 8 significant bits whose exponents lie within 13 of one another add up in fp32 without rounding
// (8 + 13 + 3 bits), and below 2^125 without passing the largest float, so that one double-double addition takes all eight; a
// vector with a wider spread (zeros do not count: one in a thousand of normally distributed weights) or a larger magnitude takes
// eight.  The sum is exact either way.  With eight conversions and double-double additions for every vector the pass was close
// to VALU-bound: 57344 x 8192, both passes, 346.6 -> 338.2 us.
typedef unsigned short sum_u16x2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ inline void add_abs(const uint4& q, dd (&part)[4], int slot) {
    const uint32_t u[4] = {q.x, q.y, q.z, q.w};
    if (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) dd_add_double(part[e], (double)fabsf(__uint_as_float(u[e])));
        return;
    }
    sum_u16x2 top = {0, 0}, low = {0xFFFF, 0xFFFF};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const sum_u16x2 mag = __builtin_bit_cast(sum_u16x2, u[e] & 0x7FFF7FFFu);
        top = __builtin_elementwise_max(top, mag);
        low = __builtin_elementwise_min(low, mag - (sum_u16x2){1, 1});           // a zero wraps to the top: it does not count
    }
    const int largest = (int)(top.x > top.y ? top.x : top.y);                    // exponents from bit 7 up
    const int widest = largest - (int)(low.x < low.y ? low.x : low.y);
    if (__builtin_expect(widest <= 12 * 128 && largest < (127 + 125) * 128, 1)) {
        float f[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[2 * e] = fabsf(__uint_as_float(u[e] << 16));
            f[2 * e + 1] = fabsf(__uint_as_float(u[e] & 0xFFFF0000u));
        }
        dd_add_double(part[slot], (double)(((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]))));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dd_add_double(part[e], (double)fabsf(__uint_as_float(u[e] << 16)));
            dd_add_double(part[e], (double)fabsf(__uint_as_float(u[e] & 0xFFFF0000u)));
        }
    }
}

// Row segments that are quantized side by side, each with a gamma of its own.  Both passes deal their workgroups out to
// the segments in proportion to the rows, so that a merged matrix takes two launches and fills the chip however it is
// divided: one pair of launches per segment ran a 9600 x 3200 fp32 matrix of three segments in 56.6 us, this in 43.7.
struct Seg {
    int64_t row0, rows;          // of W
    int64_t count;               // elements under the mean of Eq. (3)
    int64_t stream_vecs;         // 16-byte vectors of the segment that pass 1 reads with the streaming policy
    int64_t g0, nout;            // gamma_out[g0 .. g0 + nout - 1] receive the segment's gamma
    int part0, nparts;           // its partial sums; pass 1 has one workgroup for each
    int pack0, npack;            // its workgroups of pass 3
};
constexpr int kMaxSegs = 16;     // of one launch; kernels for a whole matrix take a list of one
template <int kSegs> struct SegList { int n; Seg s[kSegs]; };

// The share of thread tid of nthreads of a segment's |W| sum.
template <typename T>
__device__ __forceinline__ dd sum_abs(const T* __restrict__ W, const Seg& seg, bool vec_ok, int64_t tid, int64_t nthreads) {
    constexpr int kPer = 16 / (int)sizeof(T);             // elements per 16-byte vector
    const int64_t count = seg.count, stream_vecs = seg.stream_vecs;
    dd acc{0.0, 0.0};
    int64_t done = 0;
    if (vec_ok) {
        const int64_t nvec = count / kPer;
        const uint4* Wv = reinterpret_cast<const uint4*>(W);
        // the sums are exact, so the split into four accumulators changes nothing but the length of the dependent
        // chains; the next round of loads is requested before this round's values are added
        dd part[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
        int64_t i = tid;
        uint4 nxt[kSumLoads];
        bool have = i + (kSumLoads - 1) * nthreads < nvec;
        // The first stream_vecs vectors are read with the streaming policy (a plain read loop reaches 7.1 TB/s that
        // way against 6.4 TB/s); the end of W is read normally so that it stays in the memory-side cache, where the
        // packing pass, which starts from the end, finds it.
        auto request = [&](uint4 (&v)[kSumLoads], int64_t at) {
            if (at + (kSumLoads - 1) * nthreads < stream_vecs) {
#pragma unroll
                for (int u = 0; u < kSumLoads; ++u) v[u] = load_streaming_b128(Wv + at + u * nthreads);
            } else {
#pragma unroll
                for (int u = 0; u < kSumLoads; ++u) v[u] = Wv[at + u * nthreads];
            }
        };
        if (have) request(nxt, i);
        while (have) {
            uint4 cur[kSumLoads];
#pragma unroll
            for (int u = 0; u < kSumLoads; ++u) cur[u] = nxt[u];
            i += kSumLoads * nthreads;
            have = i + (kSumLoads - 1) * nthreads < nvec;
            if (have) request(nxt, i);
#pragma unroll
            for (int u = 0; u < kSumLoads; ++u) add_abs<T>(cur[u], part, u & 3);
        }
        for (; i < nvec; i += nthreads) add_abs<T>(Wv[i], part, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) dd_add_dd(acc, part[e]);
        done = nvec * kPer;
    }
    for (int64_t i = done + tid; i < count; i += nthreads) dd_add_double(acc, (double)fabsf(widen1(W[i])));
    return acc;
}

template <typename T, int kSegs>
__global__ __launch_bounds__(kSumThreads) void abs_sum_partials(const T* __restrict__ W_all, int64_t K, SegList<kSegs> list,
                                                                int vec_ok, double* __restrict__ partials) {
    int sg = 0;
    while (sg + 1 < list.n && (int)blockIdx.x >= list.s[sg + 1].part0) ++sg;
    const Seg& seg = list.s[sg];
    const dd acc = sum_abs(W_all + seg.row0 * K, seg, vec_ok, (int64_t)((int)blockIdx.x - seg.part0) * kSumThreads + threadIdx.x,
                           (int64_t)seg.nparts * kSumThreads);

    // fixed-shape tree over the block: the same pairs are always added in the same order
    __shared__ double sh_hi[kSumThreads];
    __shared__ double sh_lo[kSumThreads];
    sh_hi[threadIdx.x] = acc.hi;
    sh_lo[threadIdx.x] = acc.lo;
    __syncthreads();
    for (int s = kSumThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            dd a{sh_hi[threadIdx.x], sh_lo[threadIdx.x]};
            dd b{sh_hi[threadIdx.x + s], sh_lo[threadIdx.x + s]};
            dd_add_dd(a, b);
            sh_hi[threadIdx.x] = a.hi;
            sh_lo[threadIdx.x] = a.lo;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = sh_hi[0];
        partials[2 * blockIdx.x + 1] = sh_lo[0];
    }
}

// ---------------------------------------------------------------------------------------------------
// pass 2
// ---------------------------------------------------------------------------------------------------
constexpr int kFinishThreads = 256;
// The partial sums of pass 1 added up over one workgroup in a fixed tree: thread t folds partials t, t + 256, ...,
// then the 256 running pairs are halved eight times.  Returned unnormalised to every thread.
__device__ inline dd fold_partials(const double* __restrict__ partials, int nparts, double* sh_hi, double* sh_lo) {
    dd acc{0.0, 0.0};
    for (int i = threadIdx.x; i < nparts; i += kFinishThreads) {
        dd p{partials[2 * i], partials[2 * i + 1]};
        dd_add_dd(acc, p);
    }
    sh_hi[threadIdx.x] = acc.hi;
    sh_lo[threadIdx.x] = acc.lo;
    __syncthreads();
    for (int s = kFinishThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            dd a{sh_hi[threadIdx.x], sh_lo[threadIdx.x]};
            dd b{sh_hi[threadIdx.x + s], sh_lo[threadIdx.x + s]};
            dd_add_dd(a, b);
            sh_hi[threadIdx.x] = a.hi;
            sh_lo[threadIdx.x] = a.lo;
        }
        __syncthreads();
    }
    return dd{sh_hi[0], sh_lo[0]};
}

// The sum of pass 1's partials as a normalised double-double pair (hi = fl(hi + lo)): what one shard of a row-sharded
// matrix contributes to Eq. (3).  A fixed tree.
__global__ __launch_bounds__(kFinishThreads) void fold_abs_sum(const double* __restrict__ partials, int nparts,
                                                            double* __restrict__ sum) {
    __shared__ double sh_hi[kFinishThreads];
    __shared__ double sh_lo[kFinishThreads];
    const dd t = fold_partials(partials, nparts, sh_hi, sh_lo);
    if (threadIdx.x == 0) {
        const double hi = t.hi + t.lo;
        sum[0] = hi;
        sum[1] = t.lo - (hi - t.hi);                      // exact: |lo| <= |hi|
    }
}

// ---------------------------------------------------------------------------------------------------
// pass 3, 2-bit format
// ---------------------------------------------------------------------------------------------------
// One work item is a 16-row block x one 16-byte piece of a row per lane: one 1 KiB chunk of the packed layout (a K step of 256
// columns) in fp32, two in bf16.  A workgroup has four waves; wave w reads rows 4w .. 4w+3 of the item, and requests a row of its
// next item as soon as this one's has been coded.  In fp32 the four codes of a lane land in one word at bits 8 b + 2 i with i = l &
// 3, and OR-ing the four lanes of a quad completes the word, which every lane of the quad then holds; one ds_bpermute transposes
// the wave's 4 rows x 16 words so that lane 16 g + 4 t + j holds word j of quad column g for row 4w + t.  In bf16 two lanes
// complete a word; the pair holds the words of the wave's four rows twice, so the even lane hands out rows 0 and 2, the odd lane
// rows 1 and 3, and two ds_bpermute per step do the same.  The wave stores four 64-byte runs per step, no LDS memory and no barrier.
// Items are walked from the end of W backwards, workgroup b taking items b, b + gridDim.x, ...: neighbouring workgroups read
// neighbouring 1 KiB runs of the same 16 rows.
// Both passes, us, before (rows that are no whole number of 16-byte loads read element by element, loads under conditions) and now:
// bf16 28672 x 8191 408 / 182, 20000 x 5001 167 / 79, 20000 x 5004 111 / 80, 9600 x 3200 28.4 / 27.0, 57344 x 8192 342 / 340; fp32
// 20000 x 5001 167 / 145, 57344 x 8192 651 / 639.  Eight-byte loads in bf16 were slower still (57344 x 8192 496).  Two, three or six
// workgroups a CU instead of four: within 2 % but for 28672 x 8191, 197 at two and 176 at six.
constexpr int kPackThreads = 256;
constexpr int kPackBlocks = 1024;                          // four per CU

// A chunk of W of rows x cols elements, read in 16-byte pieces that lie `from` bytes behind its first element.  kAny: rows may
// start anywhere and end within a piece; the hardware takes 16-byte loads at element alignment.  Such a piece may run on into the
// next row, and one that would run out of W is read from the last 16 bytes of it: a chunk that ends early moves the bytes back and
// clears what is not its own (trimmed).  Otherwise the descriptor ends the rows.  Columns past the chunk's end are an offset out of its
// range in both.  No load depends on a condition: a wait for one of those is a wait for all that are in flight.
template <typename T, bool kAny>
struct Chunk {
    static constexpr int kE = 16 / (int)sizeof(T);         // elements of a piece
    const T* base;
    int rows, cols, lead, bytes;

    __device__ Chunk(const T* W, int64_t N, int64_t K, int64_t n0, int64_t k0, int most_rows, int most_cols) {
        const int64_t e0 = n0 * K + k0;
        rows = (int)(N - n0 < most_rows ? N - n0 : most_rows);
        cols = (int)(K - k0 < most_cols ? K - k0 : most_cols);
        lead = kAny && e0 >= kE ? 16 : 0;                  // there is always a piece in front of the end of W
        base = W + e0 - lead / (int)sizeof(T);
        const int64_t to_end = (N * K - e0) * (int64_t)sizeof(T) + lead;
        bytes = kAny ? (int)(to_end < 1 << 30 ? to_end : 1 << 30) : ((rows - 1) * (int)K + cols) * (int)sizeof(T);      // K <= 2^18
    }
    __device__ uint4 load(bool real, int from, int col) const {
        const int n = real && (!kAny || bytes >= 16) ? bytes : 0;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, n, 0x00020000 /* raw, 32-bit */);
        const int off = col < cols ? (kAny ? min(lead + from, n - 16) : from) : 1 << 30;
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 2 /* nt: the last use */));
    }
    __device__ uint4 trimmed(uint4 v, int from, int row, int col) const {
        const int moved = lead + from - min(lead + from, bytes - 16), have = row < rows ? (cols - col) * (int)sizeof(T) : 0;
        v = shift_down16(v, moved);
        uint64_t lo = (uint64_t)v.y << 32 | v.x, hi = (uint64_t)v.w << 32 | v.z;
        if (have < 16) hi = have > 8 ? hi & ~(~0ull << (8 * (have - 8))) : 0;
        if (have < 8) lo = have > 0 ? lo & ~(~0ull << (8 * have)) : 0;
        return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
    // a matrix of less than one piece: its elements one by one
    __device__ uint4 by_element(const T* W, int K, int row, int col) const {
        uint32_t u[4] = {0, 0, 0, 0};
#pragma unroll 1
        for (int e = 0; e < kE && row < rows && col + e < cols; ++e) {
            uint32_t bits;
            if constexpr (sizeof(T) == 2) bits = (uint32_t)W[row * K + col + e] << (16 * (e & 1));
            else bits = __float_as_uint(W[row * K + col + e]);
#pragma unroll
            for (int h = 0; h < 4; ++h) u[h] |= h == e * (int)sizeof(T) / 4 ? bits : 0u;
        }
        return make_uint4(u[0], u[1], u[2], u[3]);
    }
};

// element e of a piece, widened
template <typename T>
__device__ inline float piece_elem(const uint32_t (&u)[4], int e) {
    if (sizeof(T) == 4) return __uint_as_float(u[e & 3]);
    return __uint_as_float(e & 1 ? u[e >> 1] & 0xFFFF0000u : u[e >> 1] << 16);
}

// Pass 2 folded into the head of pass 3: while its first rows are on their way every workgroup adds up the partial sums of
// pass 1 (exact sums, so every workgroup gets the same bits) and takes gamma = fp32(S / (N K)), Eq. (3): one
// fp64 IEEE division, one rounding to fp32.  The segment's first workgroup writes it out, once per 16-row block of it.
__device__ inline float pack_gamma(const double* __restrict__ partials, const Seg& seg, float* __restrict__ gamma_out,
                                   double* sh_hi, double* sh_lo) {
    dd part{0.0, 0.0};
    partials += 2 * (int64_t)seg.part0;
    for (int i = threadIdx.x; i < seg.nparts; i += kPackThreads) dd_add_dd(part, dd{partials[2 * i], partials[2 * i + 1]});
    const double S = block_sum_dd<kPackThreads / kWave>(part, sh_hi, sh_lo);
    const float g = (float)(S / (double)seg.count);
    if ((int)blockIdx.x == seg.pack0)
        for (int64_t o = threadIdx.x; o < seg.nout; o += kPackThreads) gamma_out[seg.g0 + o] = g;
    return g;
}
// The magnitude from which a weight's code is +-1.
__device__ inline float pack_threshold(const double* __restrict__ partials, const Seg& seg, float* __restrict__ gamma_out,
                                       double* sh_hi, double* sh_lo) {
    const float d = pack_gamma(partials, seg, gamma_out, sh_hi, sh_lo) + kEps;      // gamma + eps, one fp32 add (Eq. (1))
    return ternary_threshold(d);                           // |w| >= thr  <=>  RoundClip(w / d) = +-1
}

// What the walk over the items of a segment does with the weights between two thresholds (guess_pack_2bit).
struct NoGuess { static constexpr bool kOn = false; };

// The items of one workgroup.  threshold() is called once, with the first rows on their way.  A segment's rows become row blocks row0 / 16
// ... of a packed matrix of RB row blocks in all (segments start on row blocks).
template <typename T, bool kAny, typename Threshold, typename Guess>
__device__ __forceinline__ void pack_items_2bit(const T* __restrict__ W, const Seg& seg, int64_t K, int64_t Kq /* quads per row */, int64_t RB,
                                       uint32_t* __restrict__ packed, const Threshold& threshold, Guess& guess) {
    constexpr int kE = 16 / (int)sizeof(T), kCols = kWave * kE, kSteps = kCols / 256;      // of an item
    const int64_t N = seg.rows, rb_off = seg.row0 / kRowsPerBlock;
    const int stride = seg.npack;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6, col = lane * kE;
    const int per_row = (int)ceil_div(K, kCols);
    const int items = (int)ceil_div(N, kRowsPerBlock) * per_row;      // N K < 2^40: below 2^29
    auto chunk = [&](int item) {
        const int it = items - 1 - item, rb = it / per_row;
        return Chunk<T, kAny>(W, N, K, (int64_t)rb * kRowsPerBlock, (int64_t)(it - rb * per_row) * kCols, kRowsPerBlock, kCols);
    };
    int from[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) from[t] = ((4 * w + t) * (int)K + col) * (int)sizeof(T);

    uint4 piece[4];
    int item = (int)blockIdx.x - seg.pack0;
    Chunk<T, kAny> c = chunk(item < items ? item : 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) piece[t] = c.load(item < items, from[t], col);
    const bool tiny = kAny && N * K < kE;
    if (tiny) {
#pragma unroll
        for (int t = 0; t < 4; ++t) piece[t] = c.by_element(W, (int)K, 4 * w + t, col);
    }

    const float thr = threshold();
    if constexpr (Guess::kOn) {
        if (!guess.known) return;                          // nothing to code with
    }

    const int t_out = (lane >> 2) & 3, g = lane >> 4;      // the lane stores word lane & 3 of row 4w + t_out, quad column g
    for (int nth = 0; item < items; item += stride, ++nth) {
        const bool more = item + stride < items;
        const Chunk<T, kAny> next = chunk(more ? item + stride : item);
        uint32_t word[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint4 v = piece[t];
            if (kAny && !tiny && (c.rows < kRowsPerBlock || c.cols < kCols)) v = c.trimmed(v, from[t], 4 * w + t, col);
            uint32_t code;                                 // column 4 h + b of the lane: bits 8 b + 2 h of its part of a word
            if constexpr (Guess::kOn) {
                code = guess.take(v, (uint32_t)nth << 13 | (uint32_t)(4 * w + t) << 9 | (uint32_t)col);
            } else {
                const uint32_t u[4] = {v.x, v.y, v.z, v.w};
                code = 0;
#pragma unroll
                for (int e = 0; e < kE; ++e) code |= ternary_code2_threshold(piece_elem<T>(u, e), thr) << (8 * (e & 3) + 2 * (e >> 2));
            }
            piece[t] = next.load(more, from[t], col);
            __builtin_amdgcn_sched_barrier(0);             // in this place: requested before the next row is waited for
            if (sizeof(T) == 2) {
                code <<= 4 * (lane & 1);
                word[t] = code | dpp_u32<0xB1>(code);      // lane ^ 1
            } else {
                word[t] = quad_or(code << (2 * (lane & 3)));
            }
        }
        if constexpr (Guess::kOn) {
            if (guess.full()) { c = next; continue; }      // the segment will be coded by settle_2bit
        }
        const int it = items - 1 - item, rb = it / per_row;
        const int64_t s0 = (int64_t)(it - rb * per_row) * kSteps;
#pragma unroll
        for (int q = 0; q < kSteps; ++q) {
            uint32_t out;
            if (sizeof(T) == 2) {
                const int src = (32 * q + 8 * g + 2 * (lane & 3) + (t_out & 1)) << 2;
                const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(lane & 1 ? word[1] : word[0]));
                const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(lane & 1 ? word[3] : word[2]));
                out = t_out < 2 ? lo : hi;
            } else {
                const int i = lane & 3;                    // lane 16 g + 4 t + j takes its word from lane 16 g + 4 j + t
                const int src = ((lane & 48) | (i << 2) | t_out) << 2;
                out = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(i == 0 ? word[0] : i == 1 ? word[1] : i == 2 ? word[2] : word[3]));
            }
            const int64_t s = s0 + q, nq = (Kq - 4 * s) < 4 ? (Kq - 4 * s) : 4;      // quads of this step (the last may hold fewer, or none)
            // word index inside the chunk: ((g * 16 + row) * 4 + j) with row = 4 w + t, and lane & 15 = 4 t + j
            if (g < nq) packed[quad_index_2bit(4 * s, rb + rb_off, 0, Kq, RB) * 4 + g * 64 + 16 * w + (lane & 15)] = out;
        }
        c = next;
    }
}

template <int kSegs>
__device__ inline int pack_segment(const SegList<kSegs>& list) {
    int sg = 0;
    while (sg + 1 < list.n && (int)blockIdx.x >= list.s[sg + 1].pack0) ++sg;
    return sg;
}

template <typename T, bool kAny, int kSegs>
__global__ __launch_bounds__(kPackThreads) void ternarize_pack_2bit(const T* __restrict__ W_all, int64_t K, int64_t Kq, int64_t RB,
                                                                    SegList<kSegs> list, const double* __restrict__ partials,
                                                                    float* __restrict__ gamma_out, uint32_t* __restrict__ packed) {
    __shared__ double sh_hi[kPackThreads / kWave];
    __shared__ double sh_lo[kPackThreads / kWave];
    const Seg& seg = list.s[pack_segment(list)];
    NoGuess none;
    pack_items_2bit<T, kAny>(W_all + seg.row0 * K, seg, K, Kq, RB, packed, [&] { return pack_threshold(partials, seg, gamma_out, sh_hi, sh_lo); }, none);
}

// ---------------------------------------------------------------------------------------------------
// 2-bit format, W read once
// ---------------------------------------------------------------------------------------------------
// gamma has to be known before the first code, and is only known after the last weight: hence two reads.  But a code asks no more of it
// than on which side of a threshold T(gamma) a weight lies, and a sample of W says where T is to within a few tenths of a percent:
//   sample_abs       runs of 128 bytes, one at a random place in each of as many equal stretches of W: the mean of |W| and, from the
//                    differences of runs side by side, its standard error.  Several runs of a row, and neighbours compared with each
//                    other alone: rows or heads of different scale do not widen the bounds (with runs of 1 KiB and the spread of all
//                    of them, a deviation of 10 % between the rows of 3200 x 3200 did, by more than the notes hold; now, us, two passes /
//                    this, at 50 %: 9600 x 3200 fp32 in three segments 43.6 / 39.4, 8192 x 8192 bf16 47.4 / 42.4, 57344 x 8192 327 / 227)
//   guess_pack_2bit  reads W once: adds up |W| exactly as pass 1 does, and codes as pass 3 does with the sample's threshold.  Weights
//                    between the thresholds of its mean -+ 4 standard errors (0.15 % of normally distributed fp32 ones, of
//                    bf16 ones those of the one or no value in between; at five, where gamma lies outside once in a million times and
//                    not once in 16000, 20000 x 5001 bf16 67 / 60) are noted down.  Where the bounds are more than 2 % apart it only
//                    adds up, as pass 1
//   settle_2bit      gamma from the exact sum; if it lies between its bounds, all weights but noted ones have their codes, and of those
//                    the ones between the two thresholds (one in ten) are changed.  If it does not, or a note pad was too small, this
//                    is pass 3.
// gamma and codes are those of the two passes bit for bit, whatever the sample says.  What fails, and what it then costs (us, two passes / this):
//   * no bounds: rows whose scales spread over decades, small segments of rows that deviate by half.  The sample, and 5 to 12 us: 57344 x
//     8192 bf16 328 / 357 (coded in vain as well: 403), 8192 x 8192 47.3 / 59.5, 4096 x 8192 fp32 44.5 / 54.6
//   * a mean that hangs on a few weights that the sample missed, each tens of thousands of times the others; the pass over W is then
//     in vain: 57344 x 8192 bf16 328 / 410, 8192 x 8192 47.5 / 73.5, 22016 x 8192 fp32 240 / 278, 4096 x 8192 44.5 / 60
//   * a value right at the threshold that very many weights share: from the item on that fills a wave's pad, that wave only adds up.  Two
//     thirds of the weights there (noted to the end as well: third figure): 57344 x 8192 bf16 325 / 373 (551), 8192 x 8192 46.7 / 63 (92),
//     22016 x 8192 fp32 240 / 254 (317)
// us, two passes / this: bf16 57344 x 8192 325 / 205, 28672 x 8192 162 / 107, 20000 x 5001 74.3 / 60, 8192 x 8192 47.4 / 40.3 (where the bounds
// hold a bf16 value these take 10 % more); fp32 57344 x 8192 638 / 385, 22016 x 8192 241 / 151, 9600 x 3200 in three segments 43.6 / 38.1, 7000 x
// 4096 39.8 / 34.6, 4096 x 4096 24.8 / 26.2.  What bounds it: the
// pass runs at 0.9 of what pass 3 alone takes in bf16 (190 us for 940 + 117 MB), in fp32 13 instructions a weight and the launches
// around it (sample 5, settling 4.9 of 38).
constexpr int64_t kGuessBytesF32 = (int64_t)96 << 20, kGuessBytesBf16 = (int64_t)128 << 20;
constexpr int64_t kGuessMost = (int64_t)1 << 30;           // weights: a workgroup's notes fit its LDS
constexpr int kNotes = 3584;                               // of a workgroup: 28 KiB of LDS, four workgroups a CU
constexpr int kRunVecs = 8;                                // a run: one 16-byte load on each of eight lanes, a line of the caches

// parts of the workspace: the partial sums from its start, ...
constexpr int kGuessBlocks = kPackBlocks + kMaxSegs;
constexpr size_t kSamplesAt = sizeof(double) * 2 * kGuessBlocks;
constexpr size_t kCountsAt = kSamplesAt + sizeof(double) * 2 * (kSumBlocks + kMaxSegs);
constexpr size_t kBoundsAt = kCountsAt + sizeof(int) * kGuessBlocks;
constexpr size_t kNotesAt = 2048 * 2 * sizeof(double);
static_assert(kBoundsAt % 16 == 0 && kBoundsAt + sizeof(float) * 4 * kMaxSegs <= kNotesAt, "... samples, counts and bounds within the 32 KiB of any call, notes behind them");

template <typename T, int kSegs>
__global__ __launch_bounds__(kSumThreads) void sample_abs(const T* __restrict__ W_all, int64_t K, SegList<kSegs> list, int batches,
                                                          double* __restrict__ samples) {
    constexpr int kWaves = kSumThreads / kWave, kRuns = kWave / kRunVecs;          // runs of one load of a wave
    int sg = 0;
    while (sg + 1 < list.n && (int)blockIdx.x >= list.s[sg + 1].part0) ++sg;
    const Seg& seg = list.s[sg];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint4* Wv = reinterpret_cast<const uint4*>(W_all + seg.row0 * K);
    const int nvec = (int)(seg.count * (int64_t)sizeof(T) / 16);       // below 2^28; a run at least: the launcher asks for 2 MiB a segment
    // Every weight is as likely as any other: stretches of a fraction's length leave no end of W out, and a run that starts late runs on into
    // the next stretch.
    const double stride = (double)nvec / (double)(seg.nparts * kWaves * batches * kSumLoads * kRuns);
    double sum = 0.0, squares = 0.0;
    for (int b = 0; b < batches; ++b) {
        uint4 v[kSumLoads];
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u) {
            const int j = (((b * kSumLoads + u) * seg.nparts + (int)blockIdx.x - seg.part0) * kWaves + wave) * kRuns + lane / kRunVecs;
            uint32_t h = (uint32_t)j * 0x9E3779B1u;                    // the place of run j in its stretch of W: a hash of j
            h = (h ^ (h >> 15)) * 0x85EBCA77u;
            h ^= h >> 13;
            const int at = (int)(j * stride) + (int)__umulhi(h, (uint32_t)stride);
            v[u] = Wv[min(at, nvec - kRunVecs) + lane % kRunVecs];
        }
#pragma unroll
        for (int u = 0; u < kSumLoads; ++u) {
            const uint32_t q[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            float run = 0.0f;
#pragma unroll
            for (int e = 0; e < 16 / (int)sizeof(T); ++e) run += fabsf(piece_elem<T>(q, e));
            run += dpp_f32<0xB1>(run);                                 // the eight lanes of the run
            run += dpp_f32<0x4E>(run);
            run += dpp_f32<0x141>(run);
            const double d = (double)run - (double)dpp_f32<0x140>(run);           // against its neighbour
            sum += (double)run;
            squares += d * d;
        }
    }
    __shared__ double sh[2][kWaves];
    sum = wave_sum_f64(sum) * (1.0 / kRunVecs);                        // each run on its eight lanes, each pair on sixteen
    squares = wave_sum_f64(squares) * (0.5 / kRunVecs);
    if (lane == 0) { sh[0][wave] = sum; sh[1][wave] = squares; }
    __syncthreads();
    if (threadIdx.x < 2) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) a += sh[threadIdx.x][q];
        samples[2 * blockIdx.x + threadIdx.x] = a;
    }
}

// gamma's bounds from a segment's samples, and the samples' mean; the same bits in every workgroup.  An empty interval (x > y) where they
// say nothing.
template <typename T>
__device__ inline float3 gamma_bounds(const double* __restrict__ samples, const Seg& seg, int batches, double* sh_hi, double* sh_lo) {
    double s = 0.0, q = 0.0;
    if ((int)threadIdx.x < seg.nparts) {
        const double2 v = reinterpret_cast<const double2*>(samples)[seg.part0 + threadIdx.x];
        s = v.x;
        q = v.y;
    }
    s = wave_sum_f64(s);
    q = wave_sum_f64(q);
    if ((threadIdx.x & 63) == 0) { sh_hi[threadIdx.x >> 6] = s; sh_lo[threadIdx.x >> 6] = q; }
    __syncthreads();
    s = (sh_hi[0] + sh_hi[1]) + (sh_hi[2] + sh_hi[3]);
    q = (sh_lo[0] + sh_lo[1]) + (sh_lo[2] + sh_lo[3]);
    static_assert(kPackThreads == 4 * kWave && kSumBlocks <= kPackThreads, "one sample per thread, four waves");
    // the squared difference of two runs side by side is the variance of their sum, so that q is that of s
    const float sampled = (float)(seg.nparts * (kSumThreads / kWave) * batches * kSumLoads) * (float)(16 * kWave / sizeof(T));
    const float inv = 1.0f / sampled, mean = (float)s * inv, off = 4.0f * inv * (float)sqrt(q) + 2e-6f * mean;
    const float lo = fmaxf(mean - off, 0.0f), hi = mean + off;
    return hi <= 1.02f * lo || hi == 0.0f ? make_float3(lo, hi, mean) : make_float3(1.0f, 0.0f, mean);
}

// The threshold that weights are coded with before gamma is known.
__device__ inline float guess_threshold(const float3& b) { return (b.z + kEps) * 0.5f; }

// What guess_pack_2bit does with a piece of a row.
//
// |W| is summed exactly, as pass 1 sums it, but with a conversion and an addition per weight: magnitudes of p significant bits from
// `least` up are multiples of 2^(1 - p) of it, so that sums of them are exact in fp64 while they stay below 2^(54 - p) of it.  A lane
// adds those in [least, most) up as they are, most 2^(54 - p) / (values that the lane meets) of least, least far enough below the mean that
// about one piece in a thousand has a smaller weight that is not zero; pieces with one, or with one of `most` and more, take
// double-double additions.
// With pass 1's own additions 9600 x 3200 fp32 took 32.5 us instead of 27.4.  Four workgroups a CU need 128 registers: at 136, bf16 took 213
// instead of 190; notes whose places went through a counter in LDS cost half a microsecond each (22016 x 4096 bf16 67 / 47).
template <typename T>
struct Noting {
    static constexpr bool kOn = true;
    static constexpr int kE = 16 / (int)sizeof(T), kBits = sizeof(T) == 2 ? 8 : 24;
    bool known;                // there are bounds
    double sum;
    dd rest;
    uint32_t least, most;      // magnitudes of T as integers (bf16: the same one in both halves)
    uint32_t lo, mid, hi;      // ... from which a weight is noted, from which it is coded +-1, and from which it is no longer noted
    int room, used;            // of the wave's own pad: no counter in LDS to wait for
    uint2* pad;

    // per_lane: values that a lane adds up
    __device__ void set(const float3& b, int per_lane) {
        known = b.x <= b.y;
        // T(d) is within a few units in the last place of d / 2
        const float t[3] = {(b.x + kEps) * (0.5f - 0x1p-20f), guess_threshold(b), (b.y + kEps) * (0.5f + 0x1p-20f)};
        uint32_t at[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) at[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(sizeof(T) == 2 ? (__float_as_uint(t[i]) + 0xFFFFu) >> 16 : __float_as_uint(t[i])));
        lo = at[0];
        mid = at[1];
        hi = at[2];
        const int exponent = b.z > 0.0f && b.z < __builtin_inff() ? max((int)(__float_as_uint(b.z) >> 23), 1) : 127;      // biased, of the mean
        const int range = 54 - kBits - (32 - __builtin_clz(per_lane)), below = sizeof(T) == 2 ? 22 : range - 8;
        const int first = exponent - below, from = max(first, 1), to = from + range;
        uint32_t l = first >= 1 ? (uint32_t)from << 23 : 1u, m = (uint32_t)min(to, 255) << 23;
        if (sizeof(T) == 2) {
            l = first >= 1 ? l >> 16 : 1u;
            l |= l << 16;
            m = m >> 16 | m;
        }
        least = (uint32_t)__builtin_amdgcn_readfirstlane((int)l);
        most = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    }

    // The lane's elements whose flags are set, one of each lane a round: place and bits.  Flags of bf16 elements 0 ... 3 are bits 0, 8, 16
    // and 24, of elements 4 ... 7 the bits behind those.  LDS alone: a store in here would make every wait of the loop a wait for all
    // loads in flight.
    __device__ __forceinline__ void note(uint32_t flags, uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t place) {
        asm("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));      // registers, not an array in scratch memory that is indexed below
        for (uint64_t who = __ballot(flags != 0); who; who = __ballot(flags != 0)) {
            if (flags) {
                const int p = __ffs((int)flags) - 1, e = sizeof(T) == 2 ? (p >> 3) + 4 * (p & 1) : p, h = sizeof(T) == 2 ? e >> 1 : e;
                const uint32_t w01 = h & 1 ? b : a, w23 = h & 1 ? d : c, w = h & 2 ? w23 : w01;
                const int at = used + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0));
                if (at < room) pad[at] = make_uint2(place + e, sizeof(T) == 4 ? w : e & 1 ? w & 0xFFFF0000u : w << 16);
                flags &= flags - 1;
            }
            used += __popcll(who);
        }
    }

    // Whether the wave's pad is full.  settle_2bit will then code the segment, and nothing is noted any more.
    __device__ __forceinline__ bool full() {
        if (used > room) lo = hi;
        return used > room;
    }

    // a row's piece, its first element at `place`
    __device__ __forceinline__ uint32_t take(const uint4& v, uint32_t place) {
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
        uint32_t code = 0, flags = 0;
        bool odd;                                          // a magnitude outside [least, most) that is not zero
        double s;
        if constexpr (sizeof(T) == 4) {
            uint32_t top = 0, d[4], from_mid[4], nearest = 0xFFFFFFFFu;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t m = u[e] & 0x7FFFFFFFu;
                top = max(top, m - least);                 // smaller ones wrap to the top, zero to the first place there
                d[e] = m - lo;
                nearest = min(nearest, d[e]);
                from_mid[e] = m + (0x80000000u - mid);     // top bit: from mid on
            }
            s = ((double)fabsf(__uint_as_float(u[0])) + (double)fabsf(__uint_as_float(u[1]))) +
                ((double)fabsf(__uint_as_float(u[2])) + (double)fabsf(__uint_as_float(u[3])));
            odd = top > 0u - least || !(s < (double)__uint_as_float(most));
            // flags and signs to the tops of four bytes, from there to their bits 0 and 1
            const uint32_t one = (__builtin_amdgcn_perm(from_mid[1], from_mid[0], 0x0c0c0703u) | __builtin_amdgcn_perm(from_mid[3], from_mid[2], 0x07030c0cu)) & 0x80808080u;
            const uint32_t sign = __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0703u) | __builtin_amdgcn_perm(u[3], u[2], 0x07030c0cu);
            code = one >> 7 | (one & sign) >> 6;
            if (__ballot(nearest < hi - lo)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) flags |= (d[e] < hi - lo ? 1u : 0u) << e;
                note(flags, u[0], u[1], u[2], u[3], place);
            }
        } else {
            typedef short s16x2 __attribute__((ext_vector_type(2)));
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            // two magnitudes of 15 bits to a word: adding 2^15 - m sets a half's top bit from magnitude m on
            const uint32_t add_lo = 0x80008000u - lo * 0x10001u, add_mid = 0x80008000u - mid * 0x10001u, add_hi = 0x80008000u - hi * 0x10001u;
            uint32_t from_mid[4];
            u16x2 top = {0, 0};
            s16x2 far = {0, 0};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const uint32_t m = u[h] & 0x7FFF7FFFu;
                from_mid[h] = m + add_mid;
                const u16x2 x = __builtin_bit_cast(u16x2, m) - __builtin_bit_cast(u16x2, least);
                top = __builtin_elementwise_max(top, x);
                far = __builtin_elementwise_max(far, __builtin_bit_cast(s16x2, x));
            }
            const uint32_t zero = 0x10000u - (least & 0xFFFFu);
            odd = max((uint32_t)top.x, (uint32_t)top.y) > zero || max((int)far.x, (int)far.y) >= (int)((most & 0xFFFFu) - (least & 0xFFFFu));
            // flags and signs of elements 4 h .. 4 h + 3 to the tops of four bytes, from there to bits 2 h and 2 h + 1
            uint32_t two[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t one = __builtin_amdgcn_perm(from_mid[2 * h + 1], from_mid[2 * h], 0x07050301u) & 0x80808080u;
                two[h] = one >> 1 | (one & __builtin_amdgcn_perm(u[2 * h + 1], u[2 * h], 0x07050301u));
            }
            code = two[0] >> 6 | two[1] >> 4;
            if (lo != hi) {
                uint32_t b[4];
#pragma unroll
                for (int h = 0; h < 4; ++h) b[h] = ((u[h] & 0x7FFF7FFFu) + add_lo) & ~((u[h] & 0x7FFF7FFFu) + add_hi);
                flags = (__builtin_amdgcn_perm(b[1], b[0], 0x07050301u) >> 7 & 0x01010101u) | (__builtin_amdgcn_perm(b[3], b[2], 0x07050301u) >> 6 & 0x02020202u);
                note(flags, u[0], u[1], u[2], u[3], place);
            }
            double half[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                half[h] = (double)fabsf(__uint_as_float(u[2 * h] << 16)) + (double)fabsf(__uint_as_float(u[2 * h] & 0xFFFF0000u));
                half[h] += (double)fabsf(__uint_as_float(u[2 * h + 1] << 16)) + (double)fabsf(__uint_as_float(u[2 * h + 1] & 0xFFFF0000u));
            }
            s = half[0] + half[1];
        }
        sum += odd ? 0.0 : s;
        if (__ballot(odd) && odd) {
#pragma unroll
            for (int e = 0; e < kE; ++e) dd_add_double(rest, (double)fabsf(piece_elem<T>(u, e)));
        }
        return code;
    }
};

template <typename T, bool kAny, int kSegs>
__global__ __launch_bounds__(kPackThreads, 4) void guess_pack_2bit(const T* __restrict__ W_all, int64_t K, int64_t Kq, int64_t RB, SegList<kSegs> list,
                                                                int batches, int cap, char* __restrict__ ws, uint32_t* __restrict__ packed) {
    __shared__ double sh_hi[kPackThreads / kWave];
    __shared__ double sh_lo[kPackThreads / kWave];
    __shared__ uint2 notes[kNotes];
    __shared__ int used[kPackThreads / kWave];
    const int sg = pack_segment(list), wave = threadIdx.x >> 6;
    const Seg& seg = list.s[sg];
    constexpr int kWaves = kPackThreads / kWave;
    Noting<T> noting{false, 0.0, {0.0, 0.0}, 0, 0, 0, 0, 0, cap / kWaves, 0, notes + wave * (kNotes / kWaves)};
    pack_items_2bit<T, kAny>(W_all + seg.row0 * K, seg, K, Kq, RB, packed, [&] {
        const float3 b = gamma_bounds<T>(reinterpret_cast<const double*>(ws + kSamplesAt), seg, batches, sh_hi, sh_lo);
        if ((int)blockIdx.x == seg.pack0 && threadIdx.x == 0) reinterpret_cast<float4*>(ws + kBoundsAt)[sg] = make_float4(b.x, b.y, guess_threshold(b), 0.0f);
        const int64_t items = ceil_div(seg.rows, kRowsPerBlock) * ceil_div(K, kWave * Noting<T>::kE);
        noting.set(b, (int)ceil_div(items, seg.npack) * 4 * Noting<T>::kE);
        return 0.0f; }, noting);

    dd acc = noting.rest;
    dd_add_double(acc, noting.sum);
    // Without bounds the segment is only added up, as by pass 1, and settle_2bit codes it.  By half of the waves, eight a CU: that many read
    // fastest.
    if (!noting.known && threadIdx.x < kPackThreads / 2)
        acc = sum_abs(W_all + seg.row0 * K, seg, true, (int64_t)((int)blockIdx.x - seg.pack0) * (kPackThreads / 2) + threadIdx.x, (int64_t)seg.npack * (kPackThreads / 2));
    __syncthreads();                                       // sh_hi and sh_lo are used again
    const dd mine = wave_sum_dd(acc);
    if ((threadIdx.x & 63) == 0) { sh_hi[wave] = mine.hi; sh_lo[wave] = mine.lo; used[wave] = noting.used; }
    __syncthreads();
    int n = 0, before = 0;
    bool over = false;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
        before += q < wave ? used[q] : 0;
        n += used[q];
        over = over || used[q] > cap / kWaves;
    }
    uint2* out = reinterpret_cast<uint2*>(ws + kNotesAt) + (int64_t)blockIdx.x * cap + before;
    for (int i = threadIdx.x & (kWave - 1); i < noting.used && !over; i += kWave) out[i] = noting.pad[i];
    if (threadIdx.x == 0) {
        reinterpret_cast<int*>(ws + kCountsAt)[blockIdx.x] = over ? cap + 1 : n;
        dd t{sh_hi[0], sh_lo[0]};
#pragma unroll
        for (int q = 1; q < kWaves; ++q) dd_add_dd(t, dd{sh_hi[q], sh_lo[q]});
        double* partials = reinterpret_cast<double*>(ws);
        partials[2 * blockIdx.x] = t.hi;
        partials[2 * blockIdx.x + 1] = t.lo;
    }
}

// A workgroup settles the notes of kPads workgroups of the pass before, as each reads all partial sums and counts of its segment (with one
// 5.5 us, two 4.9, four 4.5); two workgroups a CU are as fast as four where it comes to packing after all.
constexpr int kPads = 2;
template <typename T, bool kAny, int kSegs>
__global__ __launch_bounds__(kPackThreads) void settle_2bit(const T* __restrict__ W_all, int64_t K, int64_t Kq, int64_t RB, SegList<kSegs> list, int cap,
                                                            const char* __restrict__ ws, float* __restrict__ gamma_out, uint32_t* __restrict__ packed) {
    constexpr int kCols = kWave * 16 / (int)sizeof(T);
    __shared__ double sh_hi[kPackThreads / kWave];
    __shared__ double sh_lo[kPackThreads / kWave];
    int sg = 0, block0 = 0;
    for (; sg + 1 < list.n; ++sg) {
        const int blocks = (list.s[sg].npack + kPads - 1) / kPads;
        if ((int)blockIdx.x < block0 + blocks) break;
        block0 += blocks;
    }
    const Seg& was = list.s[sg];
    Seg seg = was;
    seg.part0 = was.pack0;                                 // a partial sum per workgroup of the pass before
    seg.nparts = was.npack;
    seg.pack0 = block0;
    seg.npack = (was.npack + kPads - 1) / kPads;
    const int* counts = reinterpret_cast<const int*>(ws + kCountsAt) + was.pack0;
    // A pad's words are those of items that no other pad has.  Its first notes are on their way before it is known what for.
    constexpr int kThreads = kPackThreads / kPads, kAhead = 256 / kThreads;       // cap >= 256
    const int own = (int)threadIdx.x % kThreads, which = ((int)blockIdx.x - block0) * kPads + (int)threadIdx.x / kThreads;
    const int pad = min(which, was.npack - 1);
    const uint2* notes = reinterpret_cast<const uint2*>(ws + kNotesAt) + (int64_t)(was.pack0 + pad) * cap;
    uint2 first[kAhead];
#pragma unroll
    for (int a = 0; a < kAhead; ++a) first[a] = notes[a * kThreads + own];
    const int n = which < was.npack ? counts[pad] : 0;
    int most = 0;
    for (int i = threadIdx.x; i < was.npack; i += kPackThreads) most = max(most, counts[i]);
    const float4 b = reinterpret_cast<const float4*>(ws + kBoundsAt)[sg];
    const float gamma = pack_gamma(reinterpret_cast<const double*>(ws), seg, gamma_out, sh_hi, sh_lo), thr = ternary_threshold(gamma + kEps);
    if (__syncthreads_or(!(gamma >= b.x && gamma <= b.y) || most > cap)) {
        NoGuess none;
        pack_items_2bit<T, kAny>(W_all + seg.row0 * K, seg, K, Kq, RB, packed, [&] { return thr; }, none);
        return;
    }
    const int per_row = (int)ceil_div(K, kCols), items = (int)ceil_div(seg.rows, kRowsPerBlock) * per_row;
    auto settle = [&](const uint2& at) {
        const float w = __uint_as_float(at.y);
        if ((fabsf(w) >= thr) == (fabsf(w) >= b.z)) return;
        const int it = items - 1 - (pad + (int)(at.x >> 13) * was.npack), rb = it / per_row;
        const int64_t col = (int64_t)(it - rb * per_row) * kCols + (at.x & 511u);
        const int64_t word = 4 * quad_index_2bit(col >> 6, seg.row0 / kRowsPerBlock + rb, (int)(at.x >> 9 & 15u), Kq, RB) + (col >> 4 & 3);
        __hip_atomic_fetch_xor(packed + word, (w > 0.0f ? 1u : 3u) << code_shift((int)col & 15), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
#pragma unroll
    for (int a = 0; a < kAhead; ++a)
        if (a * kThreads + own < n) settle(first[a]);
    for (int i = kAhead * kThreads + own; i < n; i += kThreads) settle(notes[i]);
}

// ---------------------------------------------------------------------------------------------------
// pass 3, 5-trit format
// ---------------------------------------------------------------------------------------------------
// A wave takes a 1 KiB chunk of the packed layout: 16 rows x 320 columns, in 16-byte pieces of the rows (ten loads a lane in
// bf16, twenty in fp32), each piece's successor in the wave's next chunk requested as soon as the piece has been coded.  Chunks
// are walked from the end of W backwards, like the items of the 2-bit form, neighbouring waves on neighbouring columns.
//
// The digit of a weight (its code + 1) is (w > -thr) + (w >= thr): two comparisons, and with a NaN on either side 0, which is what
// rounding and clipping the quotient make of it.  gamma + eps = infinity has no threshold: there a finite weight's quotient is 0
// and an infinite one's NaN, which is the digits of w * 0 against any threshold.
// Four digits, a byte each, become the low four trits of a packed byte in one dot product with (1, 3, 9, 27); the digits of a
// quad's last 16 columns, times 81, are the other addend of its 16 bytes.  No byte passes 242, so lane 16 g + r adds the two halves
// of row r, quad g, word by word as they come from the wave's LDS tile, and the wave stores its chunk as one 1 KiB run.
//
// Both passes, us, before (a wave per chunk from the front, 4-element loads, a division per weight, gamma in a launch of its own)
// and now: bf16 57344 x 8192 458 / 340 (the bytes of both reads at 5.5 TB/s), 20000 x 5000 113 / 75, 20000 x 5001 149 / 78, 9600 x
// 3200 43.5 / 28.4, 1024 x 1024 18.8 / 9.9; fp32 57344 x 8192 682 / 656, 20000 x 5001 175 / 143, 9600 x 3200 52.5 / 44.5.
constexpr int kTritPackWaves = kPackThreads / kWave;
constexpr int kTritPackBlocks = 768;                       // three per CU: us at one, two, three, four, 20000 x 5001 bf16 108 / 84 / 78 / 78, 9600 x 3200 31.3 / 28.1 / 28.4 / 29.2
constexpr int kTritTileBytes = 64 * 32;                    // per wave: 64 quads of 16 four-trit bytes and 16 fifth digits

template <typename T, bool kAny>
__global__ __launch_bounds__(kPackThreads) void ternarize_pack_trit5(const T* __restrict__ W, int64_t K, int64_t RB, SegList<1> list,
                                                                     const double* __restrict__ partials,
                                                                     float* __restrict__ gamma_out, uint4* __restrict__ packed) {
    constexpr int kE = 16 / (int)sizeof(T);                // elements of a piece
    constexpr int kPieces = kTritStep / kE;                // of a row; five loads a lane cover 320 of them, ...
    constexpr int kRows5 = 320 / kPieces;                  // ... whole rows,
    constexpr int kGroups = kRowsPerBlock / kRows5;        // so that lanes meet the same columns again in every group of five
    constexpr int kFifth = 64 / kE;                        // a quad's pieces from here on hold its columns 64 .. 79
    typedef uint16_t __attribute__((may_alias)) lds_u16;                   // the tile is written and read in different widths
    typedef uint32_t __attribute__((may_alias)) lds_u32;
    typedef unsigned lds_u32x4 __attribute__((ext_vector_type(4), may_alias));
    __shared__ double sh_hi[kTritPackWaves];
    __shared__ double sh_lo[kTritPackWaves];
    __shared__ __attribute__((aligned(16))) uint8_t tiles[kTritPackWaves][kTritTileBytes];
    const Seg& seg = list.s[0];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int steps = (int)ceil_div(K, kTritStep);
    const int items = (int)RB * steps;                     // N K < 2^40: below 2^29
    const int stride = (int)gridDim.x * kTritPackWaves;

    int col[5], at[5], put[5];                             // of the lane's five places: first column, bytes from the chunk's start, LDS
    bool fifth[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int f = i * kWave + lane, row = f / kPieces, c = f - row * kPieces;
        const int quad = c / (80 / kE), j = c - quad * (80 / kE);
        col[i] = c * kE;
        at[i] = (int)((row * K + col[i]) * (int64_t)sizeof(T));           // K <= 2^18
        fifth[i] = j >= kFifth;
        put[i] = (quad * kRowsPerBlock + row) * 32 + (fifth[i] ? 16 + (j - kFifth) * kE : j * (kE / 4));
    }

    auto chunk = [&](int item) {
        const int it = items - 1 - item, rb = it / steps;
        return Chunk<T, kAny>(W, seg.rows, K, (int64_t)rb * kRowsPerBlock, (int64_t)(it - rb * steps) * kTritStep, kRowsPerBlock, kTritStep);
    };
    auto from = [&](int q) { return q / 5 * kRows5 * (int)K * (int)sizeof(T) + at[q % 5]; };      // piece q of the lane: bytes, row
    auto row_of = [&](int q) { return q / 5 * kRows5 + (q % 5 * kWave + lane) / kPieces; };

    uint4 piece[5 * kGroups];
    int item = (int)blockIdx.x * kTritPackWaves + wave;
    Chunk<T, kAny> c = chunk(item < items ? item : 0);
#pragma unroll
    for (int q = 0; q < 5 * kGroups; ++q) piece[q] = c.load(item < items, from(q), col[q % 5]);
    const bool tiny = kAny && seg.rows * K < kE;
    if (tiny) {
#pragma unroll
        for (int q = 0; q < 5 * kGroups; ++q) piece[q] = c.by_element(W, (int)K, row_of(q), col[q % 5]);
    }

    const float d = pack_gamma(partials, seg, gamma_out, sh_hi, sh_lo) + kEps;       // Eq. (1): gamma + eps
    const bool no_threshold = d == __builtin_inff();
    const float thr = no_threshold ? 1.0f : ternary_threshold(d);
    const float keep = no_threshold ? 0.0f : 1.0f;

    for (; item < items; item += stride) {                                 // whole waves leave; no workgroup barrier in here
        const bool more = item + stride < items;
        const Chunk<T, kAny> next = chunk(more ? item + stride : item);
        uint8_t* tile = tiles[wave];
#pragma unroll
        for (int q = 0; q < 5 * kGroups; ++q) {
            uint4 v = piece[q];
            if (kAny && !tiny && (c.rows < kRowsPerBlock || c.cols < kTritStep)) v = c.trimmed(v, from(q), row_of(q), col[q % 5]);
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
            uint32_t dg[kE / 4];
#pragma unroll
            for (int h = 0; h < kE / 4; ++h) {
                dg[h] = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const float w = piece_elem<T>(u, 4 * h + b) * keep;
                    dg[h] += (w > -thr ? 1u << (8 * b) : 0u) + (w >= thr ? 1u << (8 * b) : 0u);
                }
            }
            piece[q] = next.load(more, from(q), col[q % 5]);
            uint8_t* to = tile + put[q % 5] + q / 5 * kRows5 * 32;
            if (fifth[q % 5]) {
#pragma unroll
                for (int h = 0; h < kE / 4; ++h) reinterpret_cast<lds_u32*>(to)[h] = dg[h] * 81u;
            } else if (sizeof(T) == 2) {
                *reinterpret_cast<lds_u16*>(to) = (uint16_t)(__builtin_amdgcn_udot4(dg[0], 0x1B090301u, 0, false) |
                                                              __builtin_amdgcn_udot4(dg[kE / 4 - 1], 0x1B090301u, 0, false) << 8);
            } else {
                *to = (uint8_t)__builtin_amdgcn_udot4(dg[0], 0x1B090301u, 0, false);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");             // the tile is the wave's own: its LDS accesses complete in order
        __builtin_amdgcn_wave_barrier();
        const lds_u32x4 sum = *reinterpret_cast<const lds_u32x4*>(tile + 32 * lane) + *reinterpret_cast<const lds_u32x4*>(tile + 32 * lane + 16);
        const int it = items - 1 - item, rb = it / steps;
        packed[64 * ((int64_t)(it - rb * steps) * RB + rb) + lane] = make_uint4(sum.x, sum.y, sum.z, sum.w);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        c = next;
    }
}

// ---------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------
int quant_weights_num_partials() { return 2048; }

// 16-byte vectors of W that pass 1 reads with the streaming policy: all but the last 192 MB (the memory-side cache
// holds 256 MB; what it keeps of W is what pass 3 reads first); each of several segments keeps its share of the 192 MB
static int64_t abs_sum_stream_vecs(int64_t count, int64_t esz, double share) {
    const int64_t keep = (int64_t)(share * (double)(((int64_t)192 << 20) / 16));
    const int64_t nvec = count * esz / 16;
    return nvec > keep ? nvec - keep : 0;
}

static int abs_sum_blocks(int64_t count, double share) {
    const int64_t want = ceil_div(count, (int64_t)kSumThreads * 16), most = (int64_t)(share * kSumBlocks + 0.5);
    const int64_t b = want < most ? want : most;
    return (int)(b < 1 ? 1 : b);
}

static int pack_blocks(int64_t rows, int64_t K, double share) {
    const int64_t items = ceil_div(rows, kRowsPerBlock) * ceil_div(K, 256), most = (int64_t)(share * kPackBlocks + 0.5);
    const int64_t b = items < most ? items : most;
    return (int)(b < 1 ? 1 : b);
}

// the segments seg_rows[0 .. n-1] that follow one another from row row0 of a matrix of K columns, n <= kSegs
template <int kSegs>
static SegList<kSegs> make_segs(const int64_t* seg_rows, int n, int64_t row0, int64_t K, int64_t esz) {
    SegList<kSegs> list{};
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += seg_rows[i];
    int part = 0, pack = 0;
    list.n = n;
    for (int i = 0; i < n; ++i) {
        const int64_t rows = seg_rows[i];
        const double share = (double)rows / (double)total;
        const int np = abs_sum_blocks(rows * K, share), nk = pack_blocks(rows, K, share);
        list.s[i] = Seg{row0, rows, rows * K, abs_sum_stream_vecs(rows * K, esz, share), row0 / kRowsPerBlock, ceil_div(rows, kRowsPerBlock),
                        part, np, pack, nk};
        row0 += rows; part += np; pack += nk;
    }
    return list;
}
static_assert(kSumBlocks + kMaxSegs <= 2048, "the workspace holds 2048 partial sums");

template <int kSegs>
static void launch_abs_sum_partials(const void* W, bool bf16, int64_t K, const SegList<kSegs>& list, double* partials, hipStream_t stream) {
    const int vec_ok = (reinterpret_cast<uintptr_t>(W) % 16) == 0;       // a segment starts a multiple of 32 bytes further on
    const dim3 grid((unsigned)(list.s[list.n - 1].part0 + list.s[list.n - 1].nparts)), block(kSumThreads);
    if (bf16) hipLaunchKernelGGL((abs_sum_partials<uint16_t, kSegs>), grid, block, 0, stream, static_cast<const uint16_t*>(W), K, list, vec_ok, partials);
    else      hipLaunchKernelGGL((abs_sum_partials<float, kSegs>), grid, block, 0, stream, static_cast<const float*>(W), K, list, vec_ok, partials);
}

// A workgroup's notes for a matrix of `count` weights: one weight in 128 and some, three times what normally distributed ones need, up to
// 3584 (one in 293 at 2^30, 1.5 times what one bf16 value next to the threshold takes).
static int guess_cap(int64_t count) {
    const int64_t want = count / kPackBlocks / 128 + 256;
    return (int)(want < kNotes ? want : kNotes) / 4 * 4;       // as much for each of its waves
}
static_assert(kGuessBytesBf16 / 2 >= kGuessBytesF32 / 4, "the query, which is not told the type, answers for fp32");
size_t quant_weights_workspace_bytes(int64_t N, int64_t K) {
    const int64_t count = N * K;
    return count * 4 >= kGuessBytesF32 && count <= kGuessMost ? kNotesAt + (size_t)kGuessBlocks * guess_cap(count) * sizeof(uint2) : kNotesAt;
}
// Whether the segments of a launch are read once.  Each needs a sample: 2 MiB of it at least.
// The pass that reads once has most to do for each item, and the lanes of an item past the row's end do it in vain: the fewer of them are
// filled, the larger a matrix has to be (us, two passes / once; share of lanes filled that breaks even at 105 MB of fp32 0.75, at 420 MB
// 0.35, of bf16 at 136 MB 0.87, at 419 MB 0.42).  fp32, K = 64 (0.25) 54.5 / 71.2 at 105 MB and 196 / 228 at 420, 192 (0.75) 37.3 / 37.3
// and 140 / 98 (96, 0.38, still loses at 420: 158 / 162); bf16, 256 (0.5) 57.1 / 71.9 at 136 MB and 154 / 142 at 419, 1280 (0.83) 49.5 / 52.2 and 146 / 102, 4100 (0.89)
// 54.0 / 50.9 and 154 / 110.
template <int kSegs>
static bool guess_applies(const void* W, int64_t N, int64_t K, int64_t esz, const SegList<kSegs>& list, size_t workspace_bytes) {
    int64_t rows = 0, row_blocks = 0;
    for (int i = 0; i < list.n; ++i) {
        rows += list.s[i].rows;
        row_blocks += ceil_div(list.s[i].rows, kRowsPerBlock);
        if (list.s[i].count * esz < (int64_t)2 << 20) return false;
    }
    const int64_t bytes = rows * K * esz, least = esz == 2 ? kGuessBytesBf16 : kGuessBytesF32, cols = kWave * 16 / esz;       // of an item
    const double filled = (double)(rows * K) / (double)(row_blocks * kRowsPerBlock * ceil_div(K, cols) * cols);
    return bytes >= least && (filled - 0.2) * (double)bytes >= 0.7 * (double)least && N * K <= kGuessMost && reinterpret_cast<uintptr_t>(W) % 16 == 0 &&
           workspace_bytes >= quant_weights_workspace_bytes(N, K);
}

hipError_t launch_abs_sum(const void* W, bool bf16, int64_t N, int64_t K, double* sum, void* workspace, hipStream_t stream) {
    double* partials = static_cast<double*>(workspace);
    const SegList<1> list = make_segs<1>(&N, 1, 0, K, bf16 ? 2 : 4);
    launch_abs_sum_partials(W, bf16, K, list, partials, stream);
    hipLaunchKernelGGL(fold_abs_sum, dim3(1), dim3(kFinishThreads), 0, stream, partials, list.s[0].nparts, sum);
    return hipGetLastError();
}

int quant_weights_max_sums() { return kPackThreads; }

// pass 3 over the segments of a packed matrix of RB row blocks
template <int kSegs>
static void launch_pack(const void* W, bool bf16, int64_t K, int64_t RB, const SegList<kSegs>& list, const double* partials, void* packed,
                        float* gamma, hipStream_t stream) {
    const bool any = K % (bf16 ? 8 : 4) != 0 || reinterpret_cast<uintptr_t>(W) % 16 != 0;       // a segment starts a multiple of 32 bytes further on
    const int64_t Kq = ceil_div(K, kColsPerQuad);
    const dim3 grid((unsigned)(list.s[list.n - 1].pack0 + list.s[list.n - 1].npack)), block(kPackThreads);
    uint32_t* out = static_cast<uint32_t*>(packed);
#define PACK(T_, A_) hipLaunchKernelGGL((ternarize_pack_2bit<T_, A_, kSegs>), grid, block, 0, stream, static_cast<const T_*>(W), K, Kq, RB, list, \
                                        partials, gamma, out)
    if (bf16) { if (any) PACK(uint16_t, true); else PACK(uint16_t, false); }
    else { if (any) PACK(float, true); else PACK(float, false); }
#undef PACK
}

// both in one: sample, guess, settle
template <int kSegs>
static void launch_guess(const void* W, bool bf16, int64_t N, int64_t K, int64_t RB, const SegList<kSegs>& list, void* packed, float* gamma, void* workspace,
                         hipStream_t stream) {
    const int64_t Kq = ceil_div(K, kColsPerQuad), esz = bf16 ? 2 : 4;
    const bool any = K % (16 / esz) != 0;
    const Seg& last = list.s[list.n - 1];
    const dim3 sgrid((unsigned)(last.part0 + last.nparts)), grid((unsigned)(last.pack0 + last.npack));
    int settling = 0;
    for (int i = 0; i < list.n; ++i) settling += (list.s[i].npack + kPads - 1) / kPads;
    // 8 MiB of samples per 256 MiB of W, 8 at least and 24 at most: 1 in 37 of 940 MB.  Eight take 3.3 us of a pass; what closer bounds save is
    // notes (in fp32 7 % of a pass at eight per 128 MiB; in bf16 10 %, where a value lies between the bounds).
    const int64_t want = (((last.row0 + last.rows - list.s[0].row0) * K * esz) + ((int64_t)1 << 27)) >> 28;
    const int batches = (int)(want < 1 ? 1 : want > 3 ? 3 : want), cap = guess_cap(N * K);
    char* ws = static_cast<char*>(workspace);
    double* samples = reinterpret_cast<double*>(ws + kSamplesAt);
    uint32_t* out = static_cast<uint32_t*>(packed);
#define GUESS(T_, A_) \
    hipLaunchKernelGGL((sample_abs<T_, kSegs>), sgrid, dim3(kSumThreads), 0, stream, static_cast<const T_*>(W), K, list, batches, samples); \
    hipLaunchKernelGGL((guess_pack_2bit<T_, A_, kSegs>), grid, dim3(kPackThreads), 0, stream, static_cast<const T_*>(W), K, Kq, RB, list, batches, cap, ws, out); \
    hipLaunchKernelGGL((settle_2bit<T_, A_, kSegs>), dim3((unsigned)settling), dim3(kPackThreads), 0, stream, static_cast<const T_*>(W), K, Kq, RB, list, cap, ws, gamma, out)
    if (bf16) { if (any) { GUESS(uint16_t, true); } else { GUESS(uint16_t, false); } }
    else { if (any) { GUESS(float, true); } else { GUESS(float, false); } }
#undef GUESS
}

static void launch_pack_trit5(const void* W, bool bf16, int64_t K, const SegList<1>& list, const double* partials, void* packed, float* gamma,
                              hipStream_t stream) {
    const int64_t RB = ceil_div(list.s[0].rows, kRowsPerBlock), most = ceil_div(RB * ceil_div(K, kTritStep), kTritPackWaves);
    const bool any = K % (bf16 ? 8 : 4) != 0 || reinterpret_cast<uintptr_t>(W) % 16 != 0;
    const dim3 grid((unsigned)(most < kTritPackBlocks ? most : kTritPackBlocks)), block(kPackThreads);
#define PACK(T_, A_) hipLaunchKernelGGL((ternarize_pack_trit5<T_, A_>), grid, block, 0, stream, static_cast<const T_*>(W), K, RB, list, partials, gamma, \
                                        static_cast<uint4*>(packed))
    if (bf16) { if (any) PACK(uint16_t, true); else PACK(uint16_t, false); }
    else { if (any) PACK(float, true); else PACK(float, false); }
#undef PACK
}

// Eq. (1)-(3) + packing of a whole matrix
hipError_t launch_quantize_weights(const void* W, bool bf16, int64_t N, int64_t K, bool trit5, void* packed, float* gamma, void* workspace,
                                   size_t workspace_bytes, hipStream_t stream) {
    double* partials = static_cast<double*>(workspace);
    SegList<1> list = make_segs<1>(&N, 1, 0, K, bf16 ? 2 : 4);
    list.s[0].nout = 1;
    if (!trit5 && guess_applies(W, N, K, bf16 ? 2 : 4, list, workspace_bytes)) {
        launch_guess(W, bf16, N, K, ceil_div(N, kRowsPerBlock), list, packed, gamma, workspace, stream);
        return hipGetLastError();
    }
    launch_abs_sum_partials(W, bf16, K, list, partials, stream);
    if (trit5) launch_pack_trit5(W, bf16, K, list, partials, packed, gamma, stream);
    else launch_pack(W, bf16, K, ceil_div(N, kRowsPerBlock), list, partials, packed, gamma, stream);
    return hipGetLastError();
}

hipError_t launch_pack_with_sums(const void* W, bool bf16, int64_t N, int64_t K, bool trit5, const double* sums, int nsums,
                                 int64_t total_count, void* packed, float* gamma, hipStream_t stream) {
    SegList<1> list = make_segs<1>(&N, 1, 0, K, bf16 ? 2 : 4);
    list.s[0].nparts = nsums;
    list.s[0].count = total_count;
    list.s[0].nout = 1;
    if (trit5) launch_pack_trit5(W, bf16, K, list, sums, packed, gamma, stream);
    else launch_pack(W, bf16, K, ceil_div(N, kRowsPerBlock), list, sums, packed, gamma, stream);
    return hipGetLastError();
}

hipError_t launch_quantize_weights_2bit_segmented(const void* W, bool bf16, int64_t N, int64_t K, const int64_t* seg_rows, int nseg,
                                                  void* packed, float* gamma_rb, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    double* partials = static_cast<double*>(workspace);
    int64_t row0 = 0;
    for (int first = 0; first < nseg; first += kMaxSegs) {               // groups use the workspace one after the other (stream order)
        const int n = nseg - first < kMaxSegs ? nseg - first : kMaxSegs;
        const SegList<kMaxSegs> list = make_segs<kMaxSegs>(seg_rows + first, n, row0, K, bf16 ? 2 : 4);
        if (guess_applies(W, N, K, bf16 ? 2 : 4, list, workspace_bytes)) {
            launch_guess(W, bf16, N, K, ceil_div(N, kRowsPerBlock), list, packed, gamma_rb, workspace, stream);
        } else {
            launch_abs_sum_partials(W, bf16, K, list, partials, stream);
            launch_pack(W, bf16, K, ceil_div(N, kRowsPerBlock), list, partials, packed, gamma_rb, stream);
        }
        for (int i = 0; i < n; ++i) row0 += seg_rows[first + i];
    }
    return hipGetLastError();
}

}  // namespace bitnet
