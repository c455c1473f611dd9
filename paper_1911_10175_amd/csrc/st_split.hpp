// fp32 products on the bf16 matrix cores without giving up fp32 accuracy, shared by the dense kernels.  Splitting a value
// into pieces of a shorter type whose products a matrix unit forms exactly is a published method (Markidis et al.,
// "NVIDIA Tensor Core Programmability, Performance & Precision", 2018; Henry, Tang and Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations", 2019: three bf16 pieces of an fp32 value).
//
// An fp32 value is the exact sum of three bf16 values (8 significant bits each, rounded to nearest, so the
// remainders carry their own sign): a = a0 + a1 + a2.  Of the nine products of two such sums the six largest
//   a0 b0, a0 b1, a1 b0, a1 b1, a0 b2, a2 b0
// are formed; the three left out are below 2^-24 of |a b| together (at most 2^-8 * 2^-17 each for two of them), and
// 5e-9 of it in the root mean square, a fifth of what rounding one fp32 product costs.  v_mfma_f32_32x32x16_bf16 does 16
// multiply-adds per element in the time v_mfma_f32_32x32x2_f32 does one, so six of them cost 6/16 of the fp32
// instruction's time per product.
//
// How the sums are taken decides the error.  v_mfma_f32_32x32x2_f32 is a chain of fused multiply-adds (measured: bit for
// bit).  v_mfma_f32_32x32x16_bf16 adds 8 products, then 8 more, each group to the accumulator with one rounding to
// nearest (16x16x32 alike: four groups of 8); within a group whatever lies 24 bits below the largest product is cut off, also of an accumulator smaller than the
// products.  With all six products on one accumulator that is twelve roundings per 16 products, of a sum that should stay
// small: a fresh accumulator for every block of the reduction (16 channels x 9 taps, or 32 x 3; 16 or 32 channels of a 1x1; 16 or 32
// pixels) joins the running sum in an fp32 addition.  Over many blocks a quarter of the fp32 instruction's error is left (2304 terms: 8.6e-7 ->
// 2.0e-7 of the norm).  Over a few blocks the accumulator is as large as the sum, and with many zeros, where fp32 instructions
// round only for the non-zero products, the error was 1.2 to 1.9 times theirs.  There the large products a0 b0 (16 bits, a
// group of them is nearly exact) go straight to the running sum, two roundings per 16 products, and only the five small ones,
// whose roundings are 2^-8 of one of the sum, have the block's accumulator (kSplitApart below; the 3x3 BWW has no registers for
// it and starts a fresh accumulator every 32 pixels, at stride 2 every 16, small products first).
//
// What is cut off leaves a small bias, which over 10^5 terms would outgrow the roundings (256->256 @56, N = 32, BWW: error
// 7.8e-7 of the norm with one sign, 2.7e-7 with both): every other block of the reduction is computed with one operand
// negated, so that the biases cancel.
//
// The values are scaled by 2^24 before they are split, so that the last bit of every fp32 value, also of a subnormal one,
// is a normal bf16 value and the decomposition is exact; the sums are scaled back by 2^-48.  Values from 2^104 and sums from
// 2^80 on become infinite or NaN that way, as infinities and NaN do by themselves (inf - inf), so exactly the outputs they
// take part in come out non-finite.  A wavefront that holds a non-finite output computes its tile again with
// v_mfma_f32_32x32x2_f32, operands straight from memory (split_redo_corr below, the redo parts of the BWW kernels), and takes
// the non-finite outputs from there.
#pragma once
#include "st_common.hpp"

namespace st {

#if defined(__HIPCC__)
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));      // MFMA operand: 8 reduction elements of one row / column
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));      // accumulator block of a 16x16 MFMA

// Operand of a reduction over pixels from a [pixel][32 channels] bf16 tile in LDS: lane l takes channel l % 32 and 8
// of the 16 pixels of the step, four per transposing read (a group of 16 lanes reads 4 pixels x 16 channels, 8 bytes
// a lane, and gets them back with a lane per channel).  p0, p1 = this lane's addresses for pixels 0-3 and 4-7 of its
// half of the step: split_tr_lane(lane) bytes into the row of the first of them.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 *LdsTr;
__device__ __forceinline__ bf16x8 split_tr_read(LdsTr p0, LdsTr p1)
{
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p0), b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p1);
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}
// channel part of a lane's address; its pixel of the four is (lane % 16) / 4
__device__ __forceinline__ int split_tr_lane(int lane) { return lane / 16 % 2 * 32 + lane % 4 * 8; }

constexpr float kSplitScale = 16777216.f;                   // 2^24
constexpr float kSplitUnscale = 1.f / (kSplitScale * kSplitScale);

// A kernel whose accumulator takes one tap or one step only issues the small products first: their sum is 2^-8 of the large ones' and
// rounds that much finer, and the roundings of the leading pieces' products remain (1x1 FWD / BWI and both BWW kernels).

// The longest reductions whose large products have the running sum for an accumulator: channel blocks of a 3x3 and of a 1x1
// correlation, pixels of a 1x1 filter gradient.  In units of half a rounding of the final sum, B blocks of T taps take 12 T + B
// with one accumulator per block, or 2 T B + B: equal at B = 6 without
// zeros, later with many; a 1x1, whose blocks of one tap join stage by stage, at 8 to 10.
// (Error of the norm with one accumulator : apart: 256 and 512 channels without zeros 2.0e-7 : 2.9e-7 and 2.1e-7 : 4.2e-7, 32
// channels with 80 % zeros 1.7e-7 : 6e-8; v_mfma_f32_32x32x2_f32 8.6e-7 on the first and 1.4e-7 on the last.)
constexpr int kSplitApart = 6, kSplitApart1x1 = 8, kSplitApartPixels = 128;

__device__ __forceinline__ void split2(float a, float b, bf16x2 &p0, bf16x2 &p1, bf16x2 &p2)
{
    floatx2 v = {a, b};
    p0 = __builtin_convertvector(v, bf16x2);
    v -= __builtin_convertvector(p0, floatx2);          // exact
    p1 = __builtin_convertvector(v, bf16x2);
    v -= __builtin_convertvector(p1, floatx2);          // exact
    p2 = __builtin_convertvector(v, bf16x2);            // exact
}

// the three pieces of four consecutive values times `scale` (kSplitScale or its negative)
__device__ __forceinline__ void split4(float4 v, float scale, bf16x4 (&p)[3])
{
    bf16x2 a[3], b[3];
    split2(v.x * scale, v.y * scale, a[0], a[1], a[2]);
    split2(v.z * scale, v.w * scale, b[0], b[1], b[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = __builtin_shufflevector(a[i], b[i], 0, 1, 2, 3);
}

__device__ __forceinline__ bool split_finite(float a) { return (__float_as_uint(a) & 0x7f800000u) != 0x7f800000u; }
__device__ __forceinline__ bool split_finite(float4 v) { return split_finite(v.x) && split_finite(v.y) && split_finite(v.z) && split_finite(v.w); }

// Between the outputs a wavefront has stored and a redo that looks at them lane by lane in another order (the kernels of 16 x 16 blocks
// store four channels of pixel lane % 16, the redo reads those of pixel lane % 32): without it neither the language nor the
// compiler orders a lane's loads behind another lane's stores.  Costs no instruction; a wavefront's accesses are performed in order
__device__ __forceinline__ void split_lanes_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- two f16 pieces of an fp32 value (long reductions: st_fwd_dense_wide.hpp says where) ----------------------------------
// a = h + l 2^-11 with h = a rounded to f16 (11 significant bits) and l = the remainder times 2^11, rounded: 23 bits and more, three
// quarters of all values exactly.  Of the four products of two such sums three are formed, h h on one accumulator, h l + l h on
// another that is 2^11 times as large: half the matrix work of the six bf16 products (v_mfma_f32_16x16x32_f16 runs at 1950 TFLOP/s on
// random operands where the bf16 one runs at 2080, and rounds alike, groups of 8; subnormal f16 operands are kept) and 4 bytes of operands a
// value instead of 6.  What is left out of a product and of the values is 7.5e-8 of it in the root mean square (5e-9 with bf16 pieces),
// but the leading pieces' accumulator takes half the roundings: over 128 reduced channels of a 3x3 and more the sum errs less.
// The method is published (Ootomo and Yokota, "Recovering single precision accuracy from Tensor Cores while surpassing the FP32
// theoretical peak performance", 2022: the remainder scaled by 2^11).
//
// f16 has 5 exponent bits, so values are scaled by a power of two.  A workgroup takes the one that puts the largest of some
// thousand of the values it will read into [2^9, 2^10), a block of 32 rows of filters, which have no outliers as a rule, into [2^11, 2^12): larger ones may be
// 64 or 16 times as large before h is infinite (such outputs come out non-finite and are computed again, as above).  From 2^-13 on, 2^22 or 2^24 below the
// largest, both pieces have all their bits.  Of a smaller value what lies below 2^-36 is lost, 2^-36 2^16 of a product at most: from 2^-14 on that is
// 2^-22 of the value, and no more is made of it.  An fp32 sum of n terms may
// be off by n 2^-24 of their magnitudes, so c values below 2^-14 are within it in outputs of 2^5 c / n and more.  Smaller outputs (twice as large, with what else is left
// out) are computed again, as above, where c is not zero: half_low counts the values a workgroup meets, the copy of the filters tells theirs.
// In normal layers one value in 2^22 (2^24) is as small as that and an output in 2^28 is smaller than 2^6 / n.  (Without the count, any output below
// 2^6 where there is one such value: 512->512 @28 345 -> 445 us with one such filter.)
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// The copy of the filters: [Ko/32][Ci/32][tap][2 pieces][2 halves of the 32 k][4 groups of 8 c][16 k][8 c] f16 (Ko padded to whole
// groups of 128), then an int per 32 produced channels, the exponent of their scale, then one per 32 produced channels and step
// (stage and tap), how many fours of its values hold one below the pieces' range, then another, which of the 32 channels have any filter there that is not zero
__host__ __device__ __forceinline__ int half_blocks(int Ko) { return (Ko + 127) / 128 * 4; }
__host__ __device__ __forceinline__ size_t half_notes(int Ko, int terms) { return (size_t)half_blocks(Ko) * 32 * terms; }      // in 4 bytes

constexpr float kHalfLow = 2048.f;                          // scale of l beside h
constexpr float kHalfSafe = 64.f;                           // times c / n: outputs from here on need no second look

// exponent of the scale that brings the largest magnitude `bits` (of a finite fp32 value; 0: nothing but zeros seen) below 2^top
constexpr int kHalfTopInput = 10, kHalfTopFilters = 12, kHalfTop = 15;       // (of samples; of all values)
constexpr int kHalfLower = 10;                              // by how much more an input's scale may be lowered for its outliers (fwd_dense_wide_body)
__device__ __forceinline__ int half_exponent(unsigned bits, int top)
{
    const int e = (int)(bits >> 23);
    return bits == 0 ? 0 : min(126 + top - max(e, 1), 116);       // (2^(e + 11), the scale of l, is finite)
}
__device__ __forceinline__ float half_scale(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }
__device__ __forceinline__ unsigned half_magnitude(float v)
{
    const unsigned b = __float_as_uint(v) & 0x7fffffffu;
    return b < 0x7f800000u ? b : 0u;
}
__device__ __forceinline__ unsigned half_magnitude(float4 v)
{
    return max(max(half_magnitude(v.x), half_magnitude(v.y)), max(half_magnitude(v.z), half_magnitude(v.w)));
}
__device__ __forceinline__ unsigned half_magnitude_or_infinite(float4 v)
{
    return max(max(__float_as_uint(v.x) & 0x7fffffffu, __float_as_uint(v.y) & 0x7fffffffu), max(__float_as_uint(v.z) & 0x7fffffffu, __float_as_uint(v.w) & 0x7fffffffu));
}
// the largest m of the wavefront's lanes
__device__ __forceinline__ unsigned wave_max(unsigned m)
{
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x111, 0xf, 0xf, false));          // row_shr 1, 2, 4, 8: lane 15 of each row
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x112, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x114, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x118, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xa, 0xf, false));          // row_bcast 15, 31: lane 63
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xc, 0xf, false));
    return (unsigned)__builtin_amdgcn_readlane((int)m, 63);
}
// magnitudes below 2^-14 of the scale 2^e, zero not among them, have keys below this one
__device__ __forceinline__ unsigned half_key(float a) { return (__float_as_uint(a) << 1) - 1u; }
__device__ __forceinline__ unsigned half_low_key(int e)
{
    const unsigned bits = e < 113 ? (unsigned)(113 - e) << 23 : 1u << (135 - e);        // of 2^(-14 - e), subnormal from e = 113 on
    return (bits << 1) - 1u;
}
// 1 if there are any among four values (counted as four)
__device__ __forceinline__ unsigned half_low(float4 v, unsigned low_key)
{
    return min(min(half_key(v.x), half_key(v.y)), min(half_key(v.z), half_key(v.w))) < low_key ? 1u : 0u;
}
// the two pieces of four consecutive values times s; low = s * kHalfLow
__device__ __forceinline__ void half4(float4 v, float s, float low, f16x4 (&p)[2])
{
    auto pair = [&](floatx2 a, f16x2 &h, f16x2 &l) __attribute__((always_inline)) {
        h = __builtin_convertvector(a * s, f16x2);
        const floatx2 r = {__builtin_fmaf((float)h[0], -kHalfLow, a[0] * low), __builtin_fmaf((float)h[1], -kHalfLow, a[1] * low)};      // exact
        l = __builtin_convertvector(r, f16x2);
    };
    f16x2 h[2], l[2];
    pair(floatx2{v.x, v.y}, h[0], l[0]);
    pair(floatx2{v.z, v.w}, h[1], l[1]);
    p[0] = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3);
    p[1] = __builtin_shufflevector(l[0], l[1], 0, 1, 2, 3);
}

// 32 pixels x 32 output channels of the correlation g once more with fp32 multiply-adds on the matrix cores: the lane's
// pixel (n, oh, ow; `valid`: it exists), output channels kb32*32 ..., channel blocks cb0 .. cb1-1 of the input.  Non-finite
// outputs in `out` are replaced.  A tap's products go to a pixel's sum only where the tap meets a sample, so padding
// never multiplies an infinite filter.  The 64 lanes of the wavefront make the call together.
// FWD / BWI of 256->256 @56, N = 8, us: 170 / 170 for ordinary values; one infinity in the input 200 / 271, in a filter
// 344 / 433, everywhere 637 / 1230.  (Output by output, each by one lane, one infinity or subnormal in the input took 9600.)
__device__ __forceinline__ void split_redo_corr(const Geom &g, const float *in, float *out, bool valid, int n, int oh, int ow,
                                                          int kb32, int cb0, int cb1)
{
    const int lane = threadIdx.x % kWave, l32 = lane % 32, half = lane / 32;
    const int CiB = g.Ci / kBlk, KoB = g.Ko / kBlk;
    const size_t plane = (size_t)g.Hi * g.Wi * kBlk;
    const int ko = min(kb32 * 32 + l32, g.Ko - 1);          // (rows past the last channel are not stored)
    const int taps = g.S * g.R;
    floatx16 sum = {};
#pragma unroll 1
    for (int tap = 0; tap < taps; ++tap) {
        const int ph = oh * g.sh - g.ph + tap / g.R, pw = ow * g.sw - g.pw + tap % g.R;
        const bool meets = valid && ph >= 0 && ph % g.uh == 0 && ph / g.uh < g.Hi && pw >= 0 && pw % g.uw == 0 && pw / g.uw < g.Wi;
        if (__ballot(meets) == 0) continue;                 // uniform
        // lanes that meet nothing read the first sample; their column is dropped
        const float *x = in + (meets ? act_off(n, cb0, ph / g.uh, pw / g.uw, CiB, g.Hi, g.Wi) : (size_t)cb0 * plane) + half * 8;
        const float *f = g.w + (g.wt ? (((size_t)cb0 * KoB + ko / kBlk) * taps + (taps - 1 - tap)) * (kBlk * kBlk) + ko % kBlk * kBlk
                                     : (((size_t)(ko / kBlk) * CiB + cb0) * taps + tap) * (kBlk * kBlk) + ko % kBlk) + half * 8 * (g.wt ? 1 : kBlk);
        const size_t fblock = (size_t)(g.wt ? KoB : 1) * taps * (kBlk * kBlk);
        floatx16 acc = {};
        float4 s[2], fv[2];
        auto load = [&]() __attribute__((always_inline)) {
            s[0] = *reinterpret_cast<const float4 *>(x);
            s[1] = *reinterpret_cast<const float4 *>(x + 4);
            if (g.wt) {
                fv[0] = *reinterpret_cast<const float4 *>(f);
                fv[1] = *reinterpret_cast<const float4 *>(f + 4);
            } else {
                fv[0] = make_float4(f[0], f[kBlk], f[2 * kBlk], f[3 * kBlk]);
                fv[1] = make_float4(f[4 * kBlk], f[5 * kBlk], f[6 * kBlk], f[7 * kBlk]);
            }
            x += plane;
            f += fblock;
        };
        load();
#pragma unroll 1
        for (int cb = cb0; cb < cb1; ++cb) {
            const float4 s0 = s[0], s1 = s[1], f0 = fv[0], f1 = fv[1];
            if (cb + 1 < cb1) load();                       // in flight during the products
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(j < 4 ? f0[j] : f1[j - 4], j < 4 ? s0[j] : s1[j - 4], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r] = meets ? sum[r] + acc[r] : sum[r];
    }
    if (!valid) return;
    // the lane's channels: 4*half + {0..3, 8..11} of each of the two 16-channel blocks
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (kb32 * 2 + b >= KoB) break;
        float *o = out + act_off(n, kb32 * 2 + b, oh, ow, KoB, g.Ho, g.Wo) + 4 * half;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (!split_finite(o[r / 4 * 8 + r % 4])) o[r / 4 * 8 + r % 4] = sum[8 * b + r];
    }
}

// The same for up to kRedoFew outputs of these 32 x 32, one by one in 64 bits, 16 channels times four taps and channel blocks at once; false, and nothing
// done, if there are more.  (Outputs that values below the pieces' range may matter to are few: 32 x 128->128 @28 BWI, one value in 10^4
// 2^-40 as large, log-normal values, all sizes between 2^-40 and 1: bf16 pieces 42 us each, fp32 multiply-adds 78, 73, 104, this 52, 47, 61.)
constexpr int kRedoFew = 8;
__device__ __forceinline__ bool split_redo_few(const Geom &g, const float *in, float *out, bool valid, int n, int oh, int ow, int kb32, int cb0, int cb1)
{
    const int lane = threadIdx.x % kWave, half = lane / 32;
    const int CiB = g.Ci / kBlk, KoB = g.Ko / kBlk, taps = g.S * g.R;
    // the lane's 16 outputs as split_redo_corr has them: channels 4*half + {0..3, 8..11} of two blocks
    auto at = [&](int i) __attribute__((always_inline)) {
        const int kb = kb32 * 2 + i / 8;
        return out + act_off(n, kb, oh, ow, KoB, g.Ho, g.Wo) + 4 * half + i % 8 / 4 * 8 + i % 4;
    };
    unsigned open = 0;
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
        if (!valid || kb32 * 2 + i / 8 >= KoB) continue;
        const float4 v = *reinterpret_cast<const float4 *>(at(i));
        open |= (split_finite(v.x) ? 0u : 1u) << i | (split_finite(v.y) ? 0u : 2u) << i | (split_finite(v.z) ? 0u : 4u) << i | (split_finite(v.w) ? 0u : 8u) << i;
    }
    int count = 0;
    for (int i = 0; i < 16; ++i) count += __popcll(__ballot((open >> i & 1) != 0));
    if (count > kRedoFew) return false;
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {
        for (unsigned long long m = __ballot((open >> i & 1) != 0); m != 0; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            const int pn = __builtin_amdgcn_readlane(n, l), poh = __builtin_amdgcn_readlane(oh, l), pow_ = __builtin_amdgcn_readlane(ow, l);
            const int k = kb32 * 32 + i / 8 * 16 + l / 32 * 4 + i % 8 / 4 * 8 + i % 4, c = lane % 16;
            double sum = 0.;
#pragma unroll 4
            for (int j = lane / 16; j < taps * (cb1 - cb0); j += 4) {
                const int tap = j % taps, cb = cb0 + j / taps;
                const int ph = poh * g.sh - g.ph + tap / g.R, pw = pow_ * g.sw - g.pw + tap % g.R;
                const bool meets = ph >= 0 && ph % g.uh == 0 && ph / g.uh < g.Hi && pw >= 0 && pw % g.uw == 0 && pw / g.uw < g.Wi;
                const float x = in[act_off(pn, cb, meets ? ph / g.uh : 0, meets ? pw / g.uw : 0, CiB, g.Hi, g.Wi) + c];
                const float f = g.w[g.wt ? (((size_t)cb * KoB + k / kBlk) * taps + (taps - 1 - tap)) * (kBlk * kBlk) + k % kBlk * kBlk + c
                                         : (((size_t)(k / kBlk) * CiB + cb) * taps + tap) * (kBlk * kBlk) + c * kBlk + k % kBlk];
                sum += meets ? (double)x * f : 0.;
            }
            for (int s = kWave / 2; s > 0; s /= 2) sum += __shfl_xor(sum, s);
            if (lane == l) *at(i) = (float)sum;
        }
    }
    return true;
}
#endif

}  // namespace st
