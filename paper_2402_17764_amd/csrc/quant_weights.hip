// Absmean ternary weight quantization (Eq. (1)-(3) of arXiv 2402.17764) for gfx950.
//
//   pass 1  abs_sum_partials : grid-stride |W| sum, double-double per thread, fixed-shape tree
//                              inside the block, one (hi, lo) pair per block into the workspace
//   pass 2                   : gamma = fp32(S / (N K)); done at the top of pass 3 (one launch and 4.5 us less)
//   pass 3  ternarize_pack   : re-reads W from its end (what pass 1 read last is still in the memory-side
//                              cache), takes the decision of Eq. (1)-(2) in fp32 and writes the packed
//                              layout one 1 KiB (row block, K step) chunk per workgroup pass
//
// The whole path is HBM-bound at 8.25 B per fp32 weight, 4.25 per bf16 one (two reads of W, one packed write).  Both reading passes
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

template <typename T, int kSegs>
__global__ __launch_bounds__(kSumThreads) void abs_sum_partials(const T* __restrict__ W_all, int64_t K, SegList<kSegs> list,
                                                                int vec_ok, double* __restrict__ partials) {
    constexpr int kPer = 16 / (int)sizeof(T);             // elements per 16-byte vector
    int sg = 0;
    while (sg + 1 < list.n && (int)blockIdx.x >= list.s[sg + 1].part0) ++sg;
    const Seg& seg = list.s[sg];
    const T* W = W_all + seg.row0 * K;
    const int64_t count = seg.rows * K, stream_vecs = seg.stream_vecs;
    dd acc{0.0, 0.0};
    const int64_t tid = (int64_t)((int)blockIdx.x - seg.part0) * kSumThreads + threadIdx.x;
    const int64_t nthreads = (int64_t)seg.nparts * kSumThreads;
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
static_assert(kSumBlocks <= kPackThreads, "the packing pass folds one partial sum of pass 1 per thread");

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
// pass 1 (one per thread; exact sums, so every workgroup gets the same bits) and takes gamma = fp32(S / (N K)), Eq. (3): one
// fp64 IEEE division, one rounding to fp32.  The segment's first workgroup writes it out, once per 16-row block of it.
__device__ inline float pack_gamma(const double* __restrict__ partials, const Seg& seg, float* __restrict__ gamma_out,
                                   double* sh_hi, double* sh_lo) {
    dd part{0.0, 0.0};
    partials += 2 * (int64_t)seg.part0;
    if ((int)threadIdx.x < seg.nparts) part = dd{partials[2 * threadIdx.x], partials[2 * threadIdx.x + 1]};
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

// A segment's rows become row blocks row0 / 16 ... of a packed matrix of RB row blocks in all (segments start on row
// blocks).
template <typename T, bool kAny, int kSegs>
__global__ __launch_bounds__(kPackThreads) void ternarize_pack_2bit(const T* __restrict__ W_all, int64_t K,
                                                                    int64_t Kq /* quads per row */, int64_t RB,
                                                                    SegList<kSegs> list, const double* __restrict__ partials,
                                                                    float* __restrict__ gamma_out, uint32_t* __restrict__ packed) {
    constexpr int kE = 16 / (int)sizeof(T), kCols = kWave * kE, kSteps = kCols / 256;      // of an item
    int sg = 0;
    while (sg + 1 < list.n && (int)blockIdx.x >= list.s[sg + 1].pack0) ++sg;
    const Seg& seg = list.s[sg];
    const T* W = W_all + seg.row0 * K;
    const int64_t N = seg.rows, rb_off = seg.row0 / kRowsPerBlock;
    const int stride = seg.npack;
    __shared__ double sh_hi[kPackThreads / kWave];
    __shared__ double sh_lo[kPackThreads / kWave];
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

    const float thr = pack_threshold(partials, seg, gamma_out, sh_hi, sh_lo);

    const int t_out = (lane >> 2) & 3, g = lane >> 4;      // the lane stores word lane & 3 of row 4w + t_out, quad column g
    for (; item < items; item += stride) {
        const bool more = item + stride < items;
        const Chunk<T, kAny> next = chunk(more ? item + stride : item);
        uint32_t word[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint4 v = piece[t];
            if (kAny && !tiny && (c.rows < kRowsPerBlock || c.cols < kCols)) v = c.trimmed(v, from[t], 4 * w + t, col);
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
            uint32_t code = 0;                             // column 4 h + b of the lane: bits 8 b + 2 h of its part of a word
#pragma unroll
            for (int e = 0; e < kE; ++e) code |= ternary_code2_threshold(piece_elem<T>(u, e), thr) << (8 * (e & 3) + 2 * (e >> 2));
            piece[t] = next.load(more, from[t], col);
            __builtin_amdgcn_sched_barrier(0);             // in this place: requested before the next row is waited for
            if (sizeof(T) == 2) {
                code <<= 4 * (lane & 1);
                word[t] = code | dpp_u32<0xB1>(code);      // lane ^ 1
            } else {
                word[t] = quad_or(code << (2 * (lane & 3)));
            }
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
                                   hipStream_t stream) {
    double* partials = static_cast<double*>(workspace);
    SegList<1> list = make_segs<1>(&N, 1, 0, K, bf16 ? 2 : 4);
    list.s[0].nout = 1;
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
                                                  void* packed, float* gamma_rb, void* workspace, hipStream_t stream) {
    double* partials = static_cast<double*>(workspace);
    int64_t row0 = 0;
    for (int first = 0; first < nseg; first += kMaxSegs) {               // groups use the workspace one after the other (stream order)
        const int n = nseg - first < kMaxSegs ? nseg - first : kMaxSegs;
        const SegList<kMaxSegs> list = make_segs<kMaxSegs>(seg_rows + first, n, row0, K, bf16 ? 2 : 4);
        launch_abs_sum_partials(W, bf16, K, list, partials, stream);
        launch_pack(W, bf16, K, ceil_div(N, kRowsPerBlock), list, partials, packed, gamma_rb, stream);
        for (int i = 0; i < n; ++i) row0 += seg_rows[first + i];
    }
    return hipGetLastError();
}

}  // namespace bitnet
