// Device-side bodies shared by the stand-alone filter-copy kernels and by the one-launch preparation of the
// self-selecting entry points (st_conv_fwd_auto / st_conv_bwi_auto): the filter copy in wavefront order that
// the zero-skipping FWD/BWI kernel reads, the copy in MFMA lane order that the dense one reads, and the zero
// count of a sample of a tensor.  All three are written for workgroups of 256 threads.
#pragma once
#include "st_common.hpp"
#include "st_split.hpp"

namespace st {

#if defined(__HIPCC__)
// The 16x16 filter blocks of all taps of (kb, cb) = `block` of the LAYER's filters w (library layout) into the
// wavefront-ordered copy wl[Ko/64][Ci][S][R][64 k] (Ko rounded up to whole groups of 64; the padding is never
// written and never used), or, with paired set, wl[Ko/128][Ci][S][R][64][2]: produced channels k and k + 64 of a
// group of 128 side by side (Ko is then a multiple of 128).  TRANSPOSE selects the BWI form (channel roles
// exchanged, taps reversed; SparseTrain Sec. 3.3).  Nine taps are loaded at a time (a workgroup per tap had one load in
// flight per thread: 512->512, both copies and the sample 18 -> 12).  tile: kWaveTile floats of LDS; with TRANSPOSE
// every thread of the workgroup must make the call.
__device__ __forceinline__ size_t wave_filters_index(int ko, int ci, int tap, int Ci, int SR, int paired)
{
    if (paired) return ((size_t)(ko / 128) * Ci + ci) * (SR * 128) + tap * 128 + (ko % kWave) * 2 + (ko / kWave) % 2;
    return ((size_t)(ko / kWave) * Ci + ci) * (SR * kWave) + tap * kWave + ko % kWave;
}


constexpr int kTapBatch = 9, kWaveTile = 2 * kTapBatch * kBlk * (kBlk + 1);
template <bool TRANSPOSE>
__device__ __forceinline__ void wave_filters_block(int block, int KB, int CB, int S, int R, const float *__restrict__ w,
                                                   float *__restrict__ wl, float *tile, int paired)
{
    const int cb = block % CB, kb = block / CB, SR = S * R;
    const int a = threadIdx.x / kBlk, b = threadIdx.x % kBlk;
    // paired: the block of the lower 64 channels of a group of 128 writes both partners, 8 contiguous bytes per
    // thread; the block of the upper 64 has nothing left to do (uniform: the whole workgroup leaves)
    if (paired && (TRANSPOSE ? cb : kb) % 8 >= 4) return;
    const float *src = w + ((size_t)kb * CB + cb) * SR * (kBlk * kBlk) + a * kBlk + b;                    // [tap][ci = a][ki = b]
    const float *src1 = src + (TRANSPOSE ? 4 : 4 * (size_t)CB) * SR * (kBlk * kBlk);                      // partner: cb + 4 or kb + 4
    // element of the copy: produced channel, reduced channel
    const int ko = TRANSPOSE ? cb * kBlk + b : kb * kBlk + b, ci = TRANSPOSE ? kb * kBlk + a : cb * kBlk + a;
    const int Ci = (TRANSPOSE ? KB : CB) * kBlk;
    auto slot = [&](int i, int partner, int row, int col) __attribute__((always_inline)) {
        return ((partner * kTapBatch + i) * kBlk + row) * (kBlk + 1) + col;
    };
    for (int t0 = 0; t0 < SR; t0 += kTapBatch) {
        float v0[kTapBatch], v1[kTapBatch];
#pragma unroll
        for (int i = 0; i < kTapBatch; ++i) {
            v0[i] = t0 + i < SR ? src[(t0 + i) * (kBlk * kBlk)] : 0.f;
            v1[i] = paired && t0 + i < SR ? src1[(t0 + i) * (kBlk * kBlk)] : 0.f;
        }
        if constexpr (TRANSPOSE) {
            if (t0 > 0) __syncthreads();
#pragma unroll
            for (int i = 0; i < kTapBatch; ++i) {
                tile[slot(i, 0, a, b)] = v0[i];
                if (paired) tile[slot(i, 1, a, b)] = v1[i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kTapBatch; ++i) {
                v0[i] = tile[slot(i, 0, b, a)];
                if (paired) v1[i] = tile[slot(i, 1, b, a)];
            }
        }
#pragma unroll
        for (int i = 0; i < kTapBatch; ++i) {
            if (t0 + i >= SR) break;
            const int tap = TRANSPOSE ? SR - 1 - (t0 + i) : t0 + i;
            float *dst = wl + wave_filters_index(ko, ci, tap, Ci, SR, paired);
            if (paired) *reinterpret_cast<float2 *>(dst) = make_float2(v0[i], v1[i]);
            else *dst = v0[i];
        }
    }
}

// Element i = 256 * block + thread of the fp32 copy the 1x1 kernel of small launches reads, [Ko/32][Ci/16][half][32 k][8 c];
// transpose and padding as below.
__device__ __forceinline__ void pw_filters_block(size_t block, int Ko, int Ci, int transpose, const float *__restrict__ w,
                                                 float *__restrict__ wd, size_t total)
{
    const size_t i = block * 256 + threadIdx.x;
    if (i >= total) return;
    const int CiB = Ci / kBlk, KoB = Ko / kBlk;
    size_t t = i;
    const int j = t % 8; t /= 8;
    const int l32 = t % 32; t /= 32;
    const int half = t % 2; t /= 2;
    const int cb = t % CiB;
    const int ko = (int)(t / CiB) * 32 + l32, ci = half * 8 + j;
    float val = 0.f;
    if (ko < Ko)
        val = transpose ? w[((size_t)cb * KoB + ko / kBlk) * (kBlk * kBlk) + (ko % kBlk) * kBlk + ci]
                        : w[((size_t)(ko / kBlk) * CiB + cb) * (kBlk * kBlk) + ci * kBlk + ko % kBlk];
    wd[i] = val;
}

// Piece i = 256 * block + thread (8 reduced channels of one produced channel and tap) of the copy in MFMA
// consumption order, [Ko/32][Ci/16][tap][3 pieces][2 halves of the 16 channels][32 k][8 c] bf16: the three bf16
// pieces of B[k][c][tap] = w[k][c][tap] (FWD); transpose = 1: the roles of the channel dimensions are swapped and the
// taps reversed (BWI).  Ko/Ci are the produced and reduced channel counts of the correlation that will consume
// the copy; produced channels are padded with zeros to a multiple of 128.  Every second group of `group` reduced channel
// blocks is negated (st_split.hpp).  total = pieces of 8.
__device__ __forceinline__ void reformat_filters_block(size_t block, int Ko, int Ci, int S, int R, int transpose, int group,
                                                       const float *__restrict__ w, float *__restrict__ wd, size_t total)
{
    const size_t i = block * 256 + threadIdx.x;
    if (i >= total) return;
    const int TAPS = S * R, CiB = Ci / kBlk, KoB = Ko / kBlk;
    size_t t = i;
    const int l32 = t % 32; t /= 32;
    const int half = t % 2; t /= 2;
    const size_t step = t;                              // (kb32 * CiB + cb) * TAPS + tap
    const int tap = t % TAPS; t /= TAPS;
    const int cb = t % CiB;
    const int kb32 = (int)(t / CiB);
    const int ko = kb32 * 32 + l32, c0 = half * 8;
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    if (ko < Ko) {
        const int v = tap / R, u = tap % R;
        if (!transpose) {
            // w[K = Ko][C = Ci]: element [ko/16][cb][v][u][ci%16][ko%16], eight of them 16 apart
            const float *p = w + ((((size_t)(ko / kBlk) * CiB + cb) * S + v) * R + u) * (kBlk * kBlk) + c0 * kBlk + ko % kBlk;
            lo = make_float4(p[0], p[kBlk], p[2 * kBlk], p[3 * kBlk]);
            hi = make_float4(p[4 * kBlk], p[5 * kBlk], p[6 * kBlk], p[7 * kBlk]);
        } else {
            // w[K = Ci][C = Ko]: element [cb][ko/16][S-1-v][R-1-u][ko%16][ci%16], eight in a row
            const float4 *p = reinterpret_cast<const float4 *>(
                w + ((((size_t)cb * KoB + ko / kBlk) * S + (S - 1 - v)) * R + (R - 1 - u)) * (kBlk * kBlk) + (ko % kBlk) * kBlk + c0);
            lo = p[0];
            hi = p[1];
        }
    }
    const float scale = cb / group % 2 ? -kSplitScale : kSplitScale;
    bf16x4 a[3], b[3];
    split4(lo, scale, a);
    split4(hi, scale, b);
    bf16x8 *out = reinterpret_cast<bf16x8 *>(wd) + step * 192 + half * 32 + l32;
#pragma unroll
    for (int q = 0; q < 3; ++q) out[q * 64] = __builtin_shufflevector(a[q], b[q], 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same for the 3x3 kernel that takes 32 reduced channels at a time and 16 produced ones (Ci a multiple of 32): [Ko/32][Ci/32][tap]
// [3 pieces][2 halves of the 32 k][4 groups of 8 c][16 k][8 c] bf16; every second group of 32 * `group` reduced channels is negated.
__device__ __forceinline__ void stage_filters_block(size_t block, int Ko, int Ci, int S, int R, int transpose, int group, const float *__restrict__ w,
                                                    float *__restrict__ wd, size_t total)
{
    const size_t i = block * 256 + threadIdx.x;
    if (i >= total) return;
    const int TAPS = S * R, CiB = Ci / kBlk, KoB = Ko / kBlk, NS = CiB / 2;
    size_t t = i;
    const int l16 = t % 16; t /= 16;
    const int grp = t % 4; t /= 4;
    const int kh = t % 2; t /= 2;
    const size_t step = t;                              // (kb32 * NS + stage) * TAPS + tap
    const int tap = t % TAPS; t /= TAPS;
    const int st = t % NS, kb = (int)(t / NS) * 2 + kh, cb = st * 2 + grp / 2, c0 = grp % 2 * 8;
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    if (kb < KoB) {
        if (!transpose) {
            // w[K = Ko][C = Ci]: element [kb][cb][tap][ci%16][ko%16], eight of them 16 apart
            const float *p = w + (((size_t)kb * CiB + cb) * TAPS + tap) * (kBlk * kBlk) + c0 * kBlk + l16;
            lo = make_float4(p[0], p[kBlk], p[2 * kBlk], p[3 * kBlk]);
            hi = make_float4(p[4 * kBlk], p[5 * kBlk], p[6 * kBlk], p[7 * kBlk]);
        } else {
            // w[K = Ci][C = Ko]: element [cb][kb][reversed tap][ko%16][ci%16], eight in a row
            const float4 *p = reinterpret_cast<const float4 *>(
                w + (((size_t)cb * KoB + kb) * TAPS + (TAPS - 1 - tap)) * (kBlk * kBlk) + l16 * kBlk + c0);
            lo = p[0];
            hi = p[1];
        }
    }
    const float scale = st / group % 2 ? -kSplitScale : kSplitScale;
    bf16x4 a[3], b[3];
    split4(lo, scale, a);
    split4(hi, scale, b);
    bf16x8 *out = reinterpret_cast<bf16x8 *>(wd) + step * 384 + kh * 64 + grp * 16 + l16;
#pragma unroll
    for (int q = 0; q < 3; ++q) out[q * 128] = __builtin_shufflevector(a[q], b[q], 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same in two f16 pieces (st_split.hpp: layout and scale).  128 threads write one step of 32 produced channels; all that write
// one of these 32 look at the same 1024 of their filters for the scale.  red: 8 unsigned of LDS; every thread of the workgroup must make the call
__device__ __forceinline__ void half_filters_block(size_t block, int Ko, int Ci, int S, int R, int transpose, const float *__restrict__ w,
                                                   float *__restrict__ wd, unsigned *red)
{
    const int TAPS = S * R, CiB = Ci / kBlk, KoB = Ko / kBlk, NS = (CiB + 1) / 2;
    const int l16 = threadIdx.x % 16, grp = threadIdx.x / 16 % 4, kh = threadIdx.x / kWave % 2;
    const size_t step = block * 2 + threadIdx.x / 128;  // (kb32 * NS + stage) * TAPS + tap: 4 blocks of 32 k, an even number
    size_t t = step;
    const int tap = t % TAPS; t /= TAPS;
    const int st = t % NS, kb32 = (int)(t / NS), kb = kb32 * 2 + kh, cb = st * 2 + grp / 2, c0 = grp % 2 * 8;
    // 16 x 16 filters of blocks b (produced) and c (reduced) of a tap of the layer's own order
    auto filters_of = [&](int b, int c, int tp) __attribute__((always_inline)) {
        return w + ((transpose ? (size_t)c * KoB + b : (size_t)b * CiB + c) * TAPS + tp) * (kBlk * kBlk);
    };
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo, sample[2] = {lo, lo};
    if (kb < KoB) {
        if (cb >= CiB) {                                // zeros beside an odd last block
        } else if (!transpose) {
            const float *p = filters_of(kb, cb, tap) + c0 * kBlk + l16;
            lo = make_float4(p[0], p[kBlk], p[2 * kBlk], p[3 * kBlk]);
            hi = make_float4(p[4 * kBlk], p[5 * kBlk], p[6 * kBlk], p[7 * kBlk]);
        } else {
            const float4 *p = reinterpret_cast<const float4 *>(filters_of(kb, cb, TAPS - 1 - tap) + l16 * kBlk + c0);
            lo = p[0];
            hi = p[1];
        }
        // evenly spaced over the reduced blocks and taps of the produced block (64 threads each of two blocks)
        const int j = grp * 16 + l16;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int at = (int)((long long)(2 * j + a) * (CiB * TAPS) / 128);
            sample[a] = reinterpret_cast<const float4 *>(filters_of(kb, at / TAPS, at % TAPS))[(j * 2 + a) * 29 % 64];
        }
    }
    const unsigned m = wave_max(max(half_magnitude(sample[0]), half_magnitude(sample[1])));
    const int wave = threadIdx.x / kWave;
    if (threadIdx.x % kWave == 0) red[wave] = m;
    __syncthreads();
    const int e = half_exponent(max(red[wave & 2], red[wave | 1]), kHalfTopFilters);
    const unsigned key = half_low_key(e);
    const unsigned lows = __popcll(__ballot(half_low(lo, key) != 0)) + __popcll(__ballot(half_low(hi, key) != 0));
    const unsigned long long filled = __ballot(lo.x != 0.f || lo.y != 0.f || lo.z != 0.f || lo.w != 0.f || hi.x != 0.f || hi.y != 0.f || hi.z != 0.f || hi.w != 0.f);
    const unsigned of_k = (unsigned)(filled | filled >> 16 | filled >> 32 | filled >> 48) & 0xffffu;
    if (threadIdx.x % kWave == 0) red[4 + wave] = lows | of_k << 16;
    __syncthreads();
    int *notes = reinterpret_cast<int *>(wd) + half_notes(Ko, NS * (2 * kBlk * TAPS));
    if (threadIdx.x % 128 == 0) {
        notes[kb32] = e;                                // (the same value from every step)
        notes[half_blocks(Ko) + step] = (int)((red[4 + wave] & 0xffffu) + (red[5 + wave] & 0xffffu));
        notes[half_blocks(Ko) * (1 + NS * TAPS) + step] = (int)(red[4 + wave] >> 16 | (red[5 + wave] & 0xffff0000u));
    }
    const float scale = st % 2 ? -half_scale(e) : half_scale(e);
    f16x4 a[2], b[2];
    half4(lo, scale, scale * kHalfLow, a);
    half4(hi, scale, scale * kHalfLow, b);
    f16x8 *out = reinterpret_cast<f16x8 *>(wd) + step * 256 + kh * 64 + grp * 16 + l16;
#pragma unroll
    for (int q = 0; q < 2; ++q) out[q * 128] = __builtin_shufflevector(a[q], b[q], 0, 1, 2, 3, 4, 5, 6, 7);
}

// Zero statistics of one tensor: the elements equal to zero in a sample of the tensor, one block of 1024
// consecutive floats out of every `stride` blocks, kSampleBlocks (64) blocks at most, 65 536 elements: enough to
// fix a zero fraction to 0.2 %.  kSampleParts (4) workgroups of 256 threads share the sample; part `part` looks
// at the sampled blocks part, part + 4, ... with all its 16 loads per thread in flight at once (one memory
// round trip, whatever the tensor size) and WRITES {zeros, elements looked at} to out[2 * part], out[2 * part + 1]:
// nothing is accumulated across workgroups, so no counter has to be cleared first and no atomics are involved;
// the readers add the four pairs (sample_zeros / sample_seen).  n is a multiple of 16 (whole channel blocks), so a float4
// lies inside the tensor or outside; the loads are made unconditionally, from the tensor's start where there is nothing to
// look at: under a condition each waited for itself, sixteen round trips one after the
// other (sample of x and dy, 80->48 @37x53, N = 3: 8.4 -> 3.9 us; its FWD, BWI and BWW together 82 -> 68).
// red: 8 unsigned of LDS.  Every thread of the workgroup must make the call.
constexpr int kSampleBlocks = 64, kSampleParts = 4;
__device__ __forceinline__ void zero_sample_block(const float *__restrict__ t, size_t n, int part, unsigned *__restrict__ out,
                                                  unsigned *red)
{
    const size_t stride = ((n + 1023) / 1024 + kSampleBlocks - 1) / kSampleBlocks, n4 = n / 4;
    constexpr int UN = kSampleBlocks / kSampleParts;
    const float4 *t4 = reinterpret_cast<const float4 *>(t);
    float4 v[UN];
#pragma unroll
    for (int i = 0; i < UN; ++i) {
        const size_t at = (size_t)(i * kSampleParts + part) * stride * 256 + threadIdx.x;
        v[i] = t4[at < n4 ? at : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
    unsigned zeros = 0, seen = 0;
#pragma unroll
    for (int i = 0; i < UN; ++i) {
        const size_t at = (size_t)(i * kSampleParts + part) * stride * 256 + threadIdx.x;
        const unsigned z = (v[i].x == 0.f ? 1u : 0u) + (v[i].y == 0.f ? 1u : 0u) + (v[i].z == 0.f ? 1u : 0u) + (v[i].w == 0.f ? 1u : 0u);
        zeros += at < n4 ? z : 0u;
        seen += at < n4 ? 4u : 0u;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        zeros += __shfl_down(zeros, off);
        seen += __shfl_down(seen, off);
    }
    if (threadIdx.x % kWave == 0) {
        red[threadIdx.x / kWave] = zeros;
        red[4 + threadIdx.x / kWave] = seen;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[2 * part] = red[0] + red[1] + red[2] + red[3];
        out[2 * part + 1] = red[4] + red[5] + red[6] + red[7];
    }
}
#endif

}  // namespace st
