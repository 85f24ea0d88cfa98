// Which launch shape of the decode kernel (decode_kernel.hpp) a fused call of one to four tokens takes.
#include "decode_kernel.hpp"

namespace bitnet {

// compiled in translation units of their own
#define EXTERN(B_, N_, P_) extern template hipError_t launch_decode<B_, N_, P_>(const DecodeForm&, const DecodeCall&)
EXTERN(true, false, false); EXTERN(false, false, false); EXTERN(true, true, false); EXTERN(false, true, false);
EXTERN(true, false, true); EXTERN(false, false, true); EXTERN(true, true, true); EXTERN(false, true, true);
#undef EXTERN

// the share of a wave's padded K walk (whole rounds of kD steps in flight) that is real steps
static double walk(int steps, int kS, int kD) { return (double)steps / (double)(kS * kD * (int)ceil_div(ceil_div(steps, kS), kD)); }

// The shapes are those of a sweep of fifteen to twenty-three per entry point over 19 ... 8192 row blocks and 2 ... 112 K steps, one,
// two and four tokens, and of one in a decoder stack (eighteen widths of 1024 ... 8192; there the norm's gain is cold and fewer,
// wider workgroups do better than alone).  What decides:
//   * up to 256 row blocks, one per workgroup, K split so that all of it is requested at once (4096 x 4096, four waves at depth 4:
//     2.97 us, eight at depth 5: 3.43; 1024 x 1536, four waves at depth 2: 2.37, eight: 2.64);
//   * then a number of row blocks per workgroup that leaves at most 256 workgroups, or as many as two per CU (5120 x 5120, two row
//     blocks on eight waves 3.86, one on four 4.06; 9600 x 8192 with the norm, four on eight waves 6.9, one on eight 7.7);
//   * short rows without a K split: nothing to fold (12288 x 512: 2.72 us, with two K waves 3.19, with four 3.25), and layers of more
//     than 1024 row blocks, where every wave has work of its own anyhow (24576 x 4096 with the norm: 6.55, two K waves 6.92);
//   * twelve row blocks per workgroup from 24 K steps on where eight would be more than 256 workgroups, as long as twelve are not (2049
//     ... 3072 row blocks; two row blocks with K split over four waves are up to 1536 workgroups that quantize the tokens each for
//     itself: 41600 x 6384 with the norm, one token 15.8 -> 14.6 us, four 42.4 -> 19.1; 48960 x 10224, one token 29.1 -> 21.8, four without
//     the norm 32.4 -> 23.2);
//   * two row blocks per wave, and so half as many workgroups that quantize, on more than 3072 row blocks: for three and four tokens
//     of up to three steps, where quantizing is most of the launch, and from 24 steps on where the workgroups then fit one round (up
//     to 4096; three and four tokens with the norm beyond that, too) (us, one row block per wave / this: 51200 x 240, four tokens 5.7 /
//     4.2; 65536 x 12288, one 35.5 / 32.9, two 36.1 / 33.5; 49280 x 10240 with the norm, three 33.7 / 25.8; 80000 x 12288, three 44.7 / 51.0);
//   * depth: whichever of the built ones pads the K walk least (27648 x 2560, ten steps: depth 5 5.04 us, depth 4 5.18).
// Between 513 and 1024 row blocks four per workgroup with K split in two are the rule, with two exceptions.  Where that split pads the
// walk by a sixth and more, and a depth of five without a split by a tenth at most, every wave walks its row block alone (8320 x 2560: 3.86 us,
// split 4.17; without the norm the longer walk costs more than the fold from 11 steps on).  And one plain token on up to 640 row
// blocks takes, for 11 to 16 steps, the shape of up to 256: four waves request all of a row block at once (10240 x 3840: 4.14 us,
// two K waves 4.40).
// The picks are within 4 % of the best measured in that sweep, most within 1 %.
// rb row blocks, steps K steps
static DecodeForm pick_rows(int64_t rb, int steps, int64_t M, bool norm) {
    if (rb <= 256) {
        if (steps <= 8) return {1, 4, 1, 2};
        if (steps <= 16) return {1, 4, 1, 4};
        const double w2 = walk(steps, 8, 2), w3 = walk(steps, 8, 3), w5 = walk(steps, 8, 5);
        return {1, 8, 1, w2 >= w3 && w2 >= w5 ? 2 : w3 >= w5 ? 3 : 5};
    }
    if (rb <= 512) {
        if (steps <= 4) return {1, 1, 4, 4};
        if (steps <= 8) return {1, 2, 2, 4};
        if (steps >= 64) return {1, 8, 2, 2};
        return {1, 4, 2, walk(steps, 4, 4) >= walk(steps, 4, 5) ? 4 : 5};
    }
    const int d = steps <= 4 || walk(steps, 1, 4) >= walk(steps, 1, 5) ? 4 : 5;
    if (rb <= 1024) {
        if (steps <= 4) return {1, 1, 4, 4};
        if (!norm && M == 1 && rb <= 640 && steps > 10 && steps <= 16) return {1, 4, 1, 4};
        if (steps <= (norm ? 20 : 10) && walk(steps, 1, 5) >= 0.9 && walk(steps, 2, 4) < 0.85) return {1, 1, 4, 5};
        return {1, 2, 4, 4};
    }
    if (rb > 3072 && steps <= 3 && M > 2) return {2, 1, 8, 2};
    if (rb > 3072 && steps >= 24 && (rb <= 4096 || (M > 2 && norm))) return {2, 1, 8, 4};
    if (rb <= 2048 || rb > 3072) return {1, 1, 8, d};
    return steps < 24 ? DecodeForm{1, 1, 4, d} : DecodeForm{1, 1, 12, 4};
}

// pairs of row blocks, the gate and the up half (one token, norm in front, us: 4096 x 1024 four K waves 3.0, none 3.3; 4096 x 4096 eight
// 3.9, four 4.1; 11008 x 2560 two pairs on eight waves 4.6, one on four 5.1; 17280 x 4096 four pairs without a split 6.2, three on
// twelve waves 6.4, one on four 6.7; 57344 x 8192 eight pairs 21.1, two on eight waves 24.6).  From 24 K steps on as many pairs per
// workgroup as make at most 256 of them, with all the K waves that leaves: three pairs on twelve waves up to 768 (17280 x 8192 9.9, one
// on eight 11.5), four beyond (32000 x 8192 12.8, three on twelve waves 17.1; 25600 x 15360 19.6 / 28.1; rows that eight waves do not
// hold, on sixteen: 32000 x 20480 29.4 / 37.3).
static DecodeForm pick_pairs(int64_t pairs, int steps, int64_t K, bool bf16) {
    const int d = steps <= 4 || walk(steps, 1, 4) >= walk(steps, 1, 5) ? 4 : 5;
    if (pairs <= 256) return steps <= 8 ? DecodeForm{2, 4, 1, 2} : DecodeForm{2, 8, 1, 2};
    if (pairs <= 512) return steps <= 4 ? DecodeForm{2, 1, 4, 4} : DecodeForm{2, 4, 2, 2};
    if (pairs > 1024) return {2, 1, 8, d};
    if (steps < 24) return {2, 1, 4, d};
    if (pairs <= 768) return {2, 4, 3, 2};
    return decode_vecs(K, 8 * kWave, bf16) <= kDecodeMaxVecs ? DecodeForm{2, 2, 4, 4} : DecodeForm{2, 4, 4, 2};
}

bool launch_decode_fused(bool bf16, bool norm, bool pair, const void* x, const float* gain, float eps, const void* packed, const float* gamma,
                         int gstride, int64_t M, int64_t N, int64_t K, void* y, OutType yt, hipStream_t stream, LaunchPlan* plan, hipError_t* status) {
    const int64_t rb = ceil_div(N, kRowsPerBlock);
    const int steps = (int)ceil_div(K, 256);
    if (M > kMaxTokens) return false;
    DecodeForm f = pair ? pick_pairs(rb, steps, K, bf16) : pick_rows(rb, steps, M, norm);
    // rows that four-wave workgroups cannot hold in registers
    if (f.s == 1 && f.w == 4 && decode_vecs(K, 256, bf16) > kDecodeMaxVecs) f.w = 8;
    const int threads = f.s * f.w * kWave, vecs = decode_vecs(K, threads, bf16);
    // three bf16 tokens with the norm that twelve or sixteen waves would hold in scratch memory: the kernel for more tokens is as fast
    if (bf16 && norm && M > 2 && (pair ? f.s * f.w == 16 : f.w == 12 && vecs > 3)) return false;
    if (vecs > kDecodeMaxVecs || decode_lds_bytes((int)M, (int)K, f.r, f.s, f.w) > 65536 ||
        ceil_div(rb, pair ? f.w : f.w * f.r) * threads >= kMaxGridThreads)
        return false;
    const DecodeCall c{x, gain, eps, packed, gamma, gstride, M, N, K, y, yt, stream, plan};
    if (pair) *status = norm ? (bf16 ? launch_decode<true, true, true>(f, c) : launch_decode<false, true, true>(f, c))
                             : (bf16 ? launch_decode<true, false, true>(f, c) : launch_decode<false, false, true>(f, c));
    else *status = norm ? (bf16 ? launch_decode<true, true, false>(f, c) : launch_decode<false, true, false>(f, c))
                        : (bf16 ? launch_decode<true, false, false>(f, c) : launch_decode<false, false, false>(f, c));
    return true;
}

}  // namespace bitnet
