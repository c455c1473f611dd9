// fp32 products on the bf16 matrix cores without giving up fp32 accuracy, shared by the dense kernels.
//
// An fp32 value is the exact sum of three bf16 values (8 significant bits each, rounded to nearest, so the
// remainders carry their own sign): a = a0 + a1 + a2.  Of the nine products of two such sums the six largest
//   a0 b0, a0 b1, a1 b0, a1 b1, a0 b2, a2 b0
// are formed; the three left out are below 2^-24 of |a b| together (at most 2^-8 * 2^-16 each for two of them), at the
// rounding of one fp32 product.  v_mfma_f32_32x32x16_bf16 does 16 multiply-adds per element in the time
// v_mfma_f32_32x32x2_f32 does one, so six of them cost 6/16 of the fp32 instruction's time per product.
//
// The matrix core adds the 16 products of an instruction to the accumulator at the accumulator's own precision,
// small terms cut off towards minus infinity rather than rounded (measured: 1 + 16 * 2^-27 returns 1).  Over a long
// reduction that is 10-20 % more error than the fp32 instruction has, and a bias that grows with the number of terms.
// Two measures take both away: the kernels start a fresh accumulator per block of the reduction (16 channels x 9
// taps, 3 where the layer has no more than 16 channels; 16 channels of a 1x1; 16 or 32 pixels) and add it to the running fp32 sum on the vector ALUs, and every other block is computed with one
// operand negated and subtracted, so that the biases cancel.  What is left is a third of the fp32 instruction's error
// in FWD / BWI (2304 terms: 6.1e-7 -> 2e-7 of the result's norm) and about half in BWW (10^5 terms: 5e-7 -> 2.7e-7).
//
// The decomposition is exact for 2^-100 <= |a| < 2^127.99: smaller values lose their last pieces below the
// smallest bf16, larger ones round to infinity.  Every element outside that range is handed to the matrix
// cores as NaN (large and infinite ones become NaN by themselves: inf - inf), so exactly the outputs it takes
// part in come out non-finite, and a kernel recomputes each non-finite output it holds with plain fp32
// multiply-adds (split_exact_* below; also the outputs that are non-finite by right).  Ordinary data never
// gets there.
#pragma once
#include "st_common.hpp"

namespace st {

#if defined(__HIPCC__)
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));      // MFMA operand: 8 reduction elements of one row / column
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

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

constexpr unsigned kSplitTiny = 0x0D800000u;        // bits of 2^-100

// NaN in place of a value the decomposition cannot carry (non-zero and below 2^-100)
__device__ __forceinline__ float split_guard(float a)
{
    const unsigned b = __float_as_uint(a) << 1;
    return b - 1u < 2u * kSplitTiny - 1u ? __uint_as_float(0x7fc00000u) : a;
}

// the same for four values at once; the common case costs six integer operations
__device__ __forceinline__ float4 split_guard4(float4 v)
{
    const unsigned a = (__float_as_uint(v.x) << 1) - 1u, b = (__float_as_uint(v.y) << 1) - 1u;
    const unsigned c = (__float_as_uint(v.z) << 1) - 1u, d = (__float_as_uint(v.w) << 1) - 1u;
    const unsigned m = min(min(a, b), min(c, d));       // zeros wrap to the largest value
    if (__builtin_expect(m < 2u * kSplitTiny - 1u, 0))
        v = make_float4(split_guard(v.x), split_guard(v.y), split_guard(v.z), split_guard(v.w));
    return v;
}

__device__ __forceinline__ void split2(float a, float b, bf16x2 &p0, bf16x2 &p1, bf16x2 &p2)
{
    floatx2 v = {a, b};
    p0 = __builtin_convertvector(v, bf16x2);
    v -= __builtin_convertvector(p0, floatx2);          // exact
    p1 = __builtin_convertvector(v, bf16x2);
    v -= __builtin_convertvector(p1, floatx2);          // exact
    p2 = __builtin_convertvector(v, bf16x2);            // exact
}

// the three pieces of four consecutive values, guarded
__device__ __forceinline__ void split4(float4 v, bf16x4 (&p)[3])
{
    v = split_guard4(v);
    bf16x2 a[3], b[3];
    split2(v.x, v.y, a[0], a[1], a[2]);
    split2(v.z, v.w, b[0], b[1], b[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = __builtin_shufflevector(a[i], b[i], 0, 1, 2, 3);
}

__device__ __forceinline__ bool split_finite(float a) { return (__float_as_uint(a) & 0x7f800000u) != 0x7f800000u; }

// One output of the correlation g (channel blocks cb0 .. cb1-1 of its input) with fp32 multiply-adds from the tensors
// themselves: g.w = the layer's filters, g.wt = BWI form (channel roles exchanged, taps reversed).
__device__ __forceinline__ float split_exact_corr(const Geom &g, const float *in, int n, int ko, int oh, int ow, int cb0, int cb1)
{
    const int CiB = g.Ci / kBlk, KoB = g.Ko / kBlk;
    float s = 0.f;
#pragma unroll 1
    for (int v = 0; v < g.S && s == s; ++v) {               // (NaN stays NaN)
        const int ph = oh * g.sh - g.ph + v;
        if (ph < 0 || ph % g.uh != 0 || ph / g.uh >= g.Hi) continue;
#pragma unroll 1
        for (int u = 0; u < g.R; ++u) {
            const int pw = ow * g.sw - g.pw + u;
            if (pw < 0 || pw % g.uw != 0 || pw / g.uw >= g.Wi) continue;
#pragma unroll 1
            for (int ci = cb0 * kBlk; ci < cb1 * kBlk && s == s; ++ci) {
                const float a = in[act_off(n, ci / kBlk, ph / g.uh, pw / g.uw, CiB, g.Hi, g.Wi) + ci % kBlk];
                const size_t blk = g.wt ? (((size_t)(ci / kBlk) * KoB + ko / kBlk) * g.S + (g.S - 1 - v)) * g.R + (g.R - 1 - u)
                                        : (((size_t)(ko / kBlk) * CiB + ci / kBlk) * g.S + v) * g.R + u;
                s = fmaf(a, g.w[blk * (kBlk * kBlk) + (g.wt ? (ko % kBlk) * kBlk + ci % kBlk : (ci % kBlk) * kBlk + ko % kBlk)], s);
            }
        }
    }
    return s;
}
#endif

}  // namespace st
