// The dense matrix-core kernel of most 3x3 correlations of 64 and more input channels (fwd_dense_wide) as a template: 32 channels
// at a time through v_mfma_f32_16x16x32_f16 (three products of two f16 pieces, HALF) or _bf16 (six of three bf16 pieces); st_split.hpp has both.
//
// Why another instruction than st_fwd_dense_impl.hpp uses: with two operands of random values in registers and nothing else to
// do, v_mfma_f32_32x32x16_bf16 runs at 1760 TFLOP/s from two wavefronts per SIMD and at 1580 from four, and
// v_mfma_f32_16x16x32_bf16 at 2080, _f16 at 1950 from either (half the accumulator traffic per product, so less power, which is what holds
// the clock down).  It rounds alike: groups of 8 products, each with one rounding of the accumulator.  Errors of the norm against 64 bits,
// half zeros: 256 channels 1.87e-7 (bf16) -> 1.4e-7 (f16), 128 1.8e-7 -> 1.2e-7, at 90 % zeros 1.4e-7 -> 1.0e-7 (BWI 1.1e-7), 95 % 1.22e-7 -> 0.98e-7 (1.23e-7 -> 1.07e-7),
// 99 % 8.7e-8 -> 8.1e-8 (8.8e-8 -> 9.0e-8: the pieces' own error is left, whatever the number of terms).  The f16 form takes a fresh
// accumulator for every 3 taps of 32 channels (9 taps: 1 % faster, error 1.6e-7).  Reductions of up to kSplitApart blocks stay on
// bf16 pieces, whose error is the smaller one there from 50 % zeros on (64 channels, 50 / 80 %: 1.06e-7 : 1.13e-7, 7.4e-8 : 1.10e-7).
//
// Wavefront = 64 pixels x 32 output channels (2 x 4 blocks of 16 x 16), workgroup = KQ column blocks x 4/KQ parts of one run of
// pixels, which share its halo.  With two wavefronts per SIMD there are registers for the next stage's samples on their way
// (loads land there while the current stage is multiplied) and LDS for a second buffer: a piece is split and written after each of
// the last taps, beside the matrix instructions, and a stage costs one barrier.  N = 32, us, bf16 pieces -> f16 pieces: 256->256 @56
// 462 -> 295 (402 TFLOP/s), 512->512 @28 485 -> 308, @14 139 -> 89, 128->128 @28 41 -> 30, stride 2 128->128 @56 46 -> 35; and on bf16 64->64 @224 533.
// What it spends its time on (256->256 @56, f16, us; parts left out in a trial, results wrong): without staging 271, without
// the stream of filters from L2 (4 GB a launch) some 30 less, without the input reads from LDS some 35 less, without all three 222; the bare
// instructions take 182.  A vector instruction beside the products costs its issue time: computing what the paths that stash have in
// common ahead of them all, where the loads are waited for, took 330, counting small values by itself 20.  Tried before: 128 pixels x
// 64 channels per workgroup, 128 x 128 with eight wavefronts, input rows at other distances in LDS (no gain).
#pragma once
#include "st_fwd_dense_impl.hpp"

namespace st {
namespace {

constexpr int kStageC = 32, kWavePx = 64;       // channels of a stage, pixels of a wavefront

// KQ = column blocks (of 32 output channels) per workgroup, HPC = samples of a halo buffer: kWideHalo for 128 output channels x 64
// pixels, kWideHaloS2 at stride 2, and with 64 output channels, where a tile has 128 pixels, kWideHalo2 (six pieces a lane) where at most a
// tenth more tiles come of it, else kWideHalo2Max (seven, and a dozen spilled registers: 64->64 @224, N = 32 535 : 547 us, 256->64 @56
// 145 : 155; but 128->64 @31x57, N = 16, where a halo of 192 samples would hold 98 pixels, 40 : 33)
// With at most 32 output channels, f16 pieces only, a tile has 256 pixels and all four wavefronts read the same filters; one buffer of 352
// samples (32 x 256->32 @56 90.2 -> 57.6 us, 10 x 512->32 @58 89.6 -> 49.0, 22 x 112->16 @165 202 -> 152; 320 samples cut some tiles short: 7 x 256->32 @123 60.5 : 85.5).
// (f16 pieces take less of LDS: 224, whole rounds of the 256 lanes; at stride 2 two buffers of 304 would fit, but ten pieces of
// staging beside nine taps spill 40 registers, 128->128 @56 35.7 : 42.4)
constexpr int kWideHalo = 160, kWideHaloS2 = 320, kWideHalo2 = 192, kWideHalo2Max = 212, kWideHalo2MaxHalf = 224, kWideHalo1 = 352;
template <int KQ, int HPC, bool HALF = false>
struct WideLds {
    static constexpr int TQ = 4 / KQ, PX = TQ * kWavePx;
    static constexpr int BUFS = HPC == kWideHaloS2 || HPC == kWideHalo1 ? 1 : 2;         // two buffers where both fit twice on a compute unit
    // pieces: [3 or 2 pieces][4 groups of 8 channels][sample][8 channels] of 16 bits, i.e. 16 bytes per sample and group,
    // so that neighbouring lanes (pixels) of an operand read are 16 bytes apart
    static constexpr int NP = HALF ? 2 : 3, BUF = HPC * 16 * NP;
    // then, HALF, for each of the four wavefronts: the largest magnitude it has met, the fours it has staged with one below the pieces' range,
    // whether outputs of it are to be computed again
    static constexpr int MISC = BUFS * BUF, FLOATS = MISC + (HALF ? 12 : 0);
    // whether there may be a second pass.  Not with one buffer: its code, though it seldom runs, has 6 to 16 more registers spilled there (32 x 256->32 @56 56.4 : 58.5 us,
    // 22 x 112->16 @165 149.6 : 156.3, stride 2 128->128 @56 34.9 : 35.2)
    static constexpr bool TWICE = HALF && BUFS == 2;
};


// wg = index of the workgroup among those of the launch, cshare = its share of the channel split; lds: WideLds::FLOATS floats, 16-byte
// aligned.  Every thread of the workgroup makes the call (the body contains barriers).
// HALF: products from two f16 pieces, else, for short reductions (kSplitApart), from three bf16 pieces.  With f16 pieces the outputs that these cannot give
// (values above their range took part, or small ones that may matter) are left to a second pass (TWICE): the first one (FIRST) returns whether any wavefront
// has such, which ones in `redo`, pixels of 16 whose outputs were zeros in `zero` (of the lane), the scale in `xe`.  The second one sets outputs of pixels that meet no value to
// zero, looks for the largest value and multiplies all over with a scale that holds it;
// where that can't help, and after it, they are computed one by one (split_redo_few) or with fp32 multiply-adds, 32 x 32 at a time, which takes five times as long as a
// whole workgroup.  us, bf16 pieces : fp32 multiply-adds only : now, one in 10^4 or 10^6 values 1000 times as large: BWI 32 x 128->128 @28 42 : 312 : 51, 42 : 176 : 47,
// 16 x 256->256 @56 253 : 993 : 257, 254 : 225 : 166, FWD 270 : 502 : 266, 258 : 195 : 173; half of the rows zero and one value in 10^4 2^-60 as large, BWI 42 : 322 : 44,
// 225 : 437 : 157.
template <int KQ, int HPC, bool HALF, int MODE, bool FIRST>
__device__ __forceinline__ bool fwd_dense_wide_body(const Geom &g, const float *__restrict__ in, const float *__restrict__ wd,
                                               float *__restrict__ out, float *__restrict__ parts, const FlatGrid &fq, int kgroups,
                                               int csplit, size_t part_stride, int wg, int cshare, int &xe, unsigned &redo, unsigned &zero, float *lds_base)
{
    using Cfg = FlatCfg<MODE>;
    using Lds = WideLds<KQ, HPC, HALF>;
    using Op = std::conditional_t<HALF, f16x8, bf16x8>;
    constexpr int NP = Lds::NP, UNITS = NP * 128;                // 16-byte units of a tap's filters
    constexpr int TAPS = 9, NT = Cfg::NT, PSTEP = Cfg::PSTEP, NV = Cfg::NV, NU = Cfg::NU;
    constexpr int NLD = (HPC * 8 + 255) / 256;                   // 16-byte pieces per lane and stage
    constexpr int NJ = HALF ? 3 : 4;                             // taps between joins (4, then 5)
    constexpr bool DB = Lds::BUFS == 2;
    static_assert(!DB || NLD <= NT, "a piece a tap");

    unsigned tid = threadIdx.x;
    if constexpr (!FIRST) asm volatile("" : "+v"(tid));         // (nothing of the first pass is kept for this one)
    // the wavefront index is the same in every lane: kept in a scalar register, and with it every tile coordinate
    const int wave = __builtin_amdgcn_readfirstlane((int)(tid / kWave)), lane = (int)(tid % kWave);
    const int l16 = lane % 16, grp = lane / 16;
    const int kqi = wave % KQ, tqi = wave / KQ;
    const int kg = wg % kgroups, tile = wg / kgroups;
    const int CiB = g.Ci / kBlk, KoB = g.Ko / kBlk, NS = (CiB + 1) / 2;      // (HALF: the last stage may have one block only)

    // strip of the tile, its columns c0 .. c0+w-1 and its pixels q0 .. of npx
    const int strip = tile % fq.strips, ti = tile / fq.strips;
    const int c0 = (int)((long long)fq.cols * strip / fq.strips), w = (int)((long long)fq.cols * (strip + 1) / fq.strips) - c0;
    const int npx = g.N * fq.rows * w, q0 = ti * fq.tpx;
    if (q0 >= npx) return false;                                 // (narrower strips have fewer tiles; uniform)
    const int qend = min(q0 + fq.tpx, npx), qs = q0 + tqi * kWavePx;
    // virtual rows: image n, grid row oh starts at n * VR + oh * PSTEP with VR = (rows-1)*PSTEP + NV
    const int VR = (fq.rows - 1) * PSTEP + NV, pitch = (w - 1) * PSTEP + NU;
    auto vrow = [&](int q) __attribute__((always_inline)) {
        const int row = q / w, n = row / fq.rows;
        return n * (NV - PSTEP) + row * PSTEP;
    };
    const int n0 = q0 / w / fq.rows, v0 = vrow(q0);
    const int used = (vrow(qend - 1) - v0 + NV) * pitch;         // samples of the halo, at most HPC

    // channel split (launches with few tiles): share 0 reduces its part of the stages into the output,
    // the others into partial outputs of their own, which sum_partials_kernel adds to it afterwards
    const int st0 = NS * cshare / csplit, st1 = NS * (cshare + 1) / csplit;
    if (cshare > 0) out = parts + (cshare - 1) * part_stride;
    const int kb32 = kg * KQ + kqi;                 // this wavefront's column block
    const bool active = kb32 * 32 < g.Ko && qs < qend;

    // sums of 2 x 16 channels times 4 x 16 pixels, and those of the current taps: of the large products with HALF, whose small ones
    // have sums of their own (`low`, 2^11 times as large), else of the small ones, while the large ones go straight to the former
    floatx4 acc[2][4], part[2][4], low[2][4];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) acc[kb][pb] = low[kb][pb] = floatx4{0.f, 0.f, 0.f, 0.f};

    // filter operand: lane supplies the pieces of element (k = kb32*32 + kb*16 + l16, c = grp*8 .. grp*8+7 of the stage) from
    // the reformatted copy: 16-byte unit ((kb32*NS + stage)*TAPS + tap)*UNITS + piece*128 + kb*64 + lane
    const Op *bbase = reinterpret_cast<const Op *>(wd) + (size_t)(active ? kb32 : 0) * NS * TAPS * UNITS;
    auto filters = [&](int step, int q, Op (&f)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) f[kb] = (bbase + (size_t)step * UNITS + q * 128 + kb * 64)[lane];
    };
    // input operand: lane supplies pixel pb*16 + l16 of its 64, channels grp*8 .. grp*8+7 of the stage
    int apix[4];
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
        const int q = min(qs + pb * 16 + l16, qend - 1);   // padding columns read a valid pixel; never stored
        apix[pb] = grp * HPC + (vrow(q) - v0) * pitch + q % w * PSTEP;
    }

    // halo staging: the 16-byte pieces of a stage, eight for a sample, are split among the 256 lanes, so that a lane's are 32 samples apart.
    // poff: the piece's pixel relative to the stage's first plane of image n0, -1 for padding
    int poff[NLD];
    const int sample0 = (int)(tid / 8), sblock = (int)(tid / 4 % 2);
    const int HW = g.Hi * g.Wi;
#pragma unroll
    for (int jj = 0; jj < NLD; ++jj) {
        const int hp = jj * 32 + sample0;
        const int vr = v0 + hp / pitch, n = vr / VR;
        const int ih = vr % VR - g.ph;
        const int iw = c0 * PSTEP + hp % pitch - g.pw;
        const bool ok = hp < used && n < g.N && ih >= 0 && ih < g.Hi && iw >= 0 && iw < g.Wi;
        poff[jj] = ok ? ((n - n0) * CiB + sblock) * HW + ih * g.Wi + iw : -1;
    }
    const size_t plane = (size_t)HW * kBlk;
    const float *in0 = in + (size_t)n0 * CiB * plane + tid % 4 * 4;
    float4 hreg[NLD];
    auto absent = [&](int st) __attribute__((always_inline)) { return HALF && 2 * st + sblock >= CiB; };
    // (unconditional loads, padding from a block of zeros: a load under a condition is waited for where the condition ends)
    auto fetch = [&](int st) __attribute__((always_inline)) {
        const float *base = in0 + 2 * st * plane;
        const bool none = absent(st);
#pragma unroll
        for (int jj = 0; jj < NLD; ++jj) {
            const float *src = poff[jj] < 0 || none ? kSplitZeros : base + (size_t)(unsigned)poff[jj] * kBlk;
            hreg[jj] = *reinterpret_cast<const float4 *>(src);
        }
    };
    float xscale = 0.f, xscale_low = 0.f;                        // HALF: of the input's pieces h and l
    unsigned low_key = 0, lows = 0;
    const int stash_at = ((sblock * 2 + (int)(tid >> 1 & 1)) * HPC + sample0) * 2 + (int)(tid & 1);
    auto stash1 = [&](char *buf, int jj) __attribute__((always_inline)) {
        if ((jj + 1) * 32 > HPC && jj * 32 + sample0 >= HPC) return;
        // (the paths that stash are many, and what they share must not be computed ahead of them all, where the loads would be waited for)
        float4 v = hreg[jj];
        asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
        if constexpr (HALF) {
            f16x4 p[2];
            half4(v, xscale, xscale_low, p);
            lows += half_low(v, low_key);
            f16x4 *dst = reinterpret_cast<f16x4 *>(buf) + stash_at + jj * 64;
#pragma unroll
            for (int i = 0; i < 2; ++i) dst[i * (8 * HPC)] = p[i];
        } else {
            bf16x4 p[3];
            split4(v, kSplitScale, p);
            bf16x4 *dst = reinterpret_cast<bf16x4 *>(buf) + stash_at + jj * 64;
#pragma unroll
            for (int i = 0; i < 3; ++i) dst[i * (8 * HPC)] = p[i];
        }
    };
    char *const lds0 = reinterpret_cast<char *>(lds_base);
    auto buffer = [&](int st) __attribute__((always_inline)) { return lds0 + (DB && (st - st0) % 2 ? Lds::BUF * 4 : 0); };

    unsigned *const misc = reinterpret_cast<unsigned *>(lds_base) + Lds::MISC;
    // (the stage's barrier comes before anyone reads it)
    auto note_lows = [&]() __attribute__((always_inline)) {
        unsigned c = 0;
        if (__ballot(lows != 0) != 0)
            for (int l = 0; l < kWave; ++l) c += (unsigned)__builtin_amdgcn_readlane((int)lows, l);
        if (lane == 0) misc[4 + wave] = c;
    };
    auto where = [&](int q, int &n, int &oh, int &ow) __attribute__((always_inline)) {
        const int row = q / w;
        n = row / fq.rows;
        oh = row % fq.rows;
        ow = c0 + q % w;
        return q < qend;
    };
    // outputs that values outside the range of the scaled pieces took part in
    auto recompute = [&]() __attribute__((always_inline)) {
        split_lanes_fence();
#pragma unroll 1
        for (int pb = 0; pb < 2; ++pb) {
            if ((redo >> pb & 1) == 0) continue;
            int n, oh, ow;
            const bool valid = where(qs + pb * 32 + lane % 32, n, oh, ow);
            if constexpr (!FIRST)
                if (split_redo_few(g, in, out, valid, n, oh, ow, kb32, 2 * st0, min(2 * st1, CiB))) continue;
            split_redo_corr(g, in, out, valid, n, oh, ow, kb32, 2 * st0, min(2 * st1, CiB));
        }
    };
    // outputs of pixels that meet no value are zeros (those of all the lane's channels were)
    unsigned empty = 0;                                          // !FIRST: such pixels, pb a bit
    auto settle = [&]() __attribute__((always_inline)) {
        const unsigned zeros = zero & empty;
        if (active && __ballot(zeros != 0) != 0) {
            bool finite[2] = {true, true};
            for (int pb = 0; pb < 4; ++pb) {
                int n, oh, ow;
                if (!where(qs + pb * 16 + l16, n, oh, ow)) continue;
                for (int kb = 0; kb < 2; ++kb) {
                    if (kb32 * 2 + kb >= KoB) continue;
                    float4 *o = reinterpret_cast<float4 *>(out + act_off(n, kb32 * 2 + kb, oh, ow, KoB, g.Ho, g.Wo) + 4 * grp);
                    if ((zeros >> pb & 1) != 0) *o = make_float4(0.f, 0.f, 0.f, 0.f);
                    else finite[pb / 2] = finite[pb / 2] && split_finite(*o);
                }
            }
            redo = (__ballot(!finite[0]) != 0 ? 1u : 0u) | (__ballot(!finite[1]) != 0 ? 2u : 0u);
        }
        if (redo != 0) recompute();
    };
    if constexpr (!FIRST) {
        // the largest value of all: whether those above the sampled ones are the reason for the second pass, and not so far above that the others
        // would be small beside them; and which samples hold any value
        unsigned *const filled = reinterpret_cast<unsigned *>(lds_base);
        if (tid < HPC) filled[tid] = 0;
        static_assert(HPC <= 256, "a sample a thread");
        unsigned m = 0, most_of[NLD] = {};
#pragma unroll 1
        for (int st = st0; st < st1; ++st) {
            fetch(st);
#pragma unroll
            for (int jj = 0; jj < NLD; ++jj) most_of[jj] = max(most_of[jj], half_magnitude_or_infinite(hreg[jj]));
        }
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < NLD; ++jj) {
            m = max(m, most_of[jj]);
            if (most_of[jj] != 0 && jj * 32 + sample0 < HPC) filled[jj * 32 + sample0] = 1;        // (the same value from every thread)
        }
        m = wave_max(m);
        if (lane == 0) misc[wave] = m;
        __syncthreads();
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            unsigned any = 0;
            static_for<0, NT>([&](auto T) __attribute__((always_inline)) { any |= filled[apix[pb] - grp * HPC + Cfg::dv(decltype(T)::value) * pitch + Cfg::du(decltype(T)::value)]; });
            if (any == 0) empty |= 1u << pb;
        }
        __syncthreads();                                         // (the samples of the second pass go there)
        const unsigned most = (unsigned)__builtin_amdgcn_readfirstlane((int)max(max(misc[0], misc[1]), max(misc[2], misc[3])));
        const int e = half_exponent(most, kHalfTop);
        if (most >= 0x7f800000u || e >= xe || xe - e > kHalfLower) {
            settle();
            return false;
        }
        xe = e;
#pragma unroll
        for (int jj = 0; jj < NLD; ++jj) asm volatile("" : "+v"(poff[jj]));           // (else addresses are kept from here on)
    }
    fetch(st0);
    Op f[NP][2];
#pragma unroll
    for (int q = 0; q < NP; ++q) filters(st0 * TAPS + Cfg::ftap(0), q, f[q]);
    if constexpr (HALF) {
        if constexpr (FIRST) {
            // the first stage and, spread over the others, a piece of each lane
            const int st = st0 + (int)((tid / 4u) % (unsigned)(st1 - st0));
            const float *src = poff[0] < 0 || absent(st) ? kSplitZeros : in0 + 2 * st * plane + (size_t)(unsigned)poff[0] * kBlk;
            unsigned m = half_magnitude(*reinterpret_cast<const float4 *>(src));
#pragma unroll
            for (int jj = 0; jj < NLD; ++jj) m = max(m, half_magnitude(hreg[jj]));
            m = wave_max(m);
            if (lane == 0) misc[wave] = m;
            __syncthreads();
            xe = __builtin_amdgcn_readfirstlane(half_exponent(max(max(misc[0], misc[1]), max(misc[2], misc[3])), kHalfTopInput));
        }
        xscale = half_scale(xe);
        xscale_low = half_scale(xe + 11);
        low_key = half_low_key(xe);
    }
#pragma unroll
    for (int jj = 0; jj < NLD; ++jj) stash1(buffer(st0), jj);
    if constexpr (HALF) note_lows();
    __syncthreads();

    // one stage; More: another one follows (the last one is compiled by itself: the staging of the next under a condition costs
    // 13 to 30 spilled registers)
    auto stage = [&](int st, auto More) __attribute__((always_inline)) {
        constexpr bool more = decltype(More)::value;
        if constexpr (more) fetch(st + 1);
        const Op *lds = reinterpret_cast<const Op *>(buffer(st));
        char *const next = buffer(st + 1);
        auto input = [&](int tp, int q, Op (&x)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) x[pb] = lds[apix[pb] + Cfg::dv(tp) * pitch + Cfg::du(tp) + q * 4 * HPC];
        };
        if (active) {
            Op x[NP][4];
            static_for<0, NP>([&](auto Q) __attribute__((always_inline)) { input(0, decltype(Q)::value, x[decltype(Q)::value]); });
            // One tap = three or six products of 2 x 4 blocks.  Every operand register is refilled for the next tap as soon as its last
            // product of this one has been issued (filter piece 0, used first and last, has a second set).  The last tap requests
            // the filters of the next stage's first one.
            static_for<0, NT>([&](auto T) __attribute__((always_inline)) {
                constexpr int tp = decltype(T)::value;
                constexpr bool last = tp + 1 == NT;
                constexpr int nt = last ? 0 : tp + 1;
                const int nstep = (last && more ? st + 1 : st) * TAPS + Cfg::ftap(nt);
                auto mul = [&](const Op (&fk)[2], const Op (&xp)[4], floatx4 (&to)[2][4], bool first) __attribute__((always_inline)) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb) {            // rows = output channels, columns = pixels
                            const floatx4 c = first ? floatx4{0.f, 0.f, 0.f, 0.f} : to[kb][pb];
                            if constexpr (HALF) to[kb][pb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fk[kb], xp[pb], c, 0, 0, 0);
                            else to[kb][pb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fk[kb], xp[pb], c, 0, 0, 0);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                };
                constexpr bool fresh = tp % NJ == 0 && tp < 8;
                Op f0n[2];
                filters(nstep, 0, f0n);
                if constexpr (HALF) {
                    mul(f[0], x[0], part, fresh);
                    mul(f[1], x[0], low, false);
                    filters(nstep, 1, f[1]);
                    if constexpr (!last) input(nt, 0, x[0]);
                    mul(f[0], x[1], low, false);
                    if constexpr (!last) input(nt, 1, x[1]);
                } else {
                    mul(f[0], x[0], acc, false);
                    mul(f[NP - 1], x[0], part, fresh);
                    filters(nstep, 2, f[NP - 1]);
                    mul(f[1], x[0], part, false);
                    if constexpr (!last) input(nt, 0, x[0]);
                    mul(f[1], x[1], part, false);
                    filters(nstep, 1, f[1]);
                    mul(f[0], x[1], part, false);
                    if constexpr (!last) input(nt, 1, x[1]);
                    mul(f[0], x[NP - 1], part, false);
                    if constexpr (!last) input(nt, 2, x[NP - 1]);
                }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) f[0][kb] = f0n[kb];
                if constexpr (DB && more && tp >= NT - NLD) stash1(next, tp - (NT - NLD));
                if constexpr ((tp + 1) % NJ == 0 && tp + 1 < 8) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb) acc[kb][pb] += part[kb][pb];
                    __builtin_amdgcn_sched_barrier(0);          // (else the next tap's products get registers of their own)
                }
            });
            // the products of the last taps join the sum, which changes sign: odd stages have their filters negated (st_split.hpp)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) {
                    acc[kb][pb] = -acc[kb][pb] - part[kb][pb];
                    if constexpr (HALF) low[kb][pb] = -low[kb][pb];
                }
        } else if (DB && more) {
#pragma unroll
            for (int jj = 0; jj < NLD; ++jj) stash1(next, jj);
        }
        if constexpr (more) {
            if constexpr (!DB) {
                __syncthreads();                        // every wavefront is done with this stage
#pragma unroll
                for (int jj = 0; jj < NLD; ++jj) stash1(next, jj);
            }
            if constexpr (HALF) if (st + 2 == st1) note_lows();
            __syncthreads();
        }
    };
    for (int st = st0; st + 1 < st1; ++st) stage(st, std::true_type{});
    stage(st1 - 1, std::false_type{});

    // D layout of a 16x16 block: column (pixel) = lane % 16, row (channel) = 4*(lane/16) + r: four consecutive channels, one
    // 16-byte store
    if (active) {
        bool finite[2] = {true, true};
        const float scale = (st1 % 2 ? -1.f : 1.f) * (HALF ? 1.f : kSplitUnscale);
        int exponent = 0;
        if constexpr (HALF) {
            const int *notes = reinterpret_cast<const int *>(wd) + half_notes(g.Ko, NS * (kStageC * TAPS));
            exponent = -(xe + notes[kb32]);
            float least = kHalfSafe;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        acc[kb][pb][r] = __builtin_fmaf(low[kb][pb][r], 1.f / kHalfLow, acc[kb][pb][r]);
                        least = fminf(least, fabsf(acc[kb][pb][r]));
                    }
            // smaller ones than this may lack what values below the pieces' range would have given, but for channels without filters, whose outputs are zeros
            if (__ballot(least < kHalfSafe) != 0) {
                unsigned c = lane < 4 ? misc[4 + lane] : 0, filled = 0;
                const int *counts = notes + half_blocks(g.Ko) + kb32 * (NS * TAPS), *channels = counts + half_blocks(g.Ko) * (NS * TAPS);
                for (int i = st0 * TAPS + lane; i < st1 * TAPS; i += kWave) {
                    c += (unsigned)counts[i];
                    filled |= (unsigned)channels[i];
                }
                if (__ballot(c != 0) != 0) {
                    unsigned sum = 0, any = 0;
                    for (int l = 0; l < kWave; ++l) {
                        sum += (unsigned)__builtin_amdgcn_readlane((int)c, l);
                        any |= (unsigned)__builtin_amdgcn_readlane((int)filled, l);
                    }
                    if constexpr (Lds::TWICE) {
                        zero = 0;
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb) {
                            bool all = true;
#pragma unroll
                            for (int i = 0; i < 8; ++i) all = all && acc[i / 4][pb][i % 4] == 0.f;
                            if (all) zero |= 1u << pb;
                        }
                    }
                    const float safe = kHalfSafe * fminf(4.f * (float)sum / (float)((st1 - st0) * (kStageC * TAPS)), 1.f);
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (fabsf(acc[kb][pb][r]) < safe && (any >> (kb * 16 + 4 * grp + r) & 1) != 0) acc[kb][pb][r] = __builtin_nanf("");
                }
            }
        }
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            int n, oh, ow;
            if (!where(qs + pb * 16 + l16, n, oh, ow)) continue;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                if (kb32 * 2 + kb >= KoB) continue;
                const floatx4 a = acc[kb][pb];
                float4 r = make_float4(a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale);
                if constexpr (HALF) r = make_float4(ldexpf(r.x, exponent), ldexpf(r.y, exponent), ldexpf(r.z, exponent), ldexpf(r.w, exponent));
                finite[pb / 2] = finite[pb / 2] && split_finite(r);
                *reinterpret_cast<float4 *>(out + act_off(n, kb32 * 2 + kb, oh, ow, KoB, g.Ho, g.Wo) + 4 * grp) = r;
            }
        }
        redo = (__ballot(!finite[0]) != 0 ? 1u : 0u) | (__ballot(!finite[1]) != 0 ? 2u : 0u);
    }
    if constexpr (Lds::TWICE && FIRST) {
        if (lane == 0) misc[8 + wave] = redo;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane((int)(misc[8] | misc[9] | misc[10] | misc[11])) != 0;
    }
    if constexpr (!FIRST) settle();
    else if (__builtin_expect(redo != 0, 0)) recompute();
    return false;
}

// The arguments of the kernel as they lie in memory
struct WideArgs {
    Geom g;
    const float *in, *wd;
    float *out, *parts;
    FlatGrid fq;
    int kgroups, csplit;
    size_t part_stride;
};

template <int KQ, int HPC, bool HALF, int MODE>
__global__ __launch_bounds__(256, 2) void fwd_dense_wide_kernel(WideArgs a)
{
    if (form_deselected(a.g.sel, a.g.want, a.g.thr)) return;
    __shared__ __attribute__((aligned(16))) float lds[WideLds<KQ, HPC, HALF>::FLOATS];
    int xe = 0;
    unsigned redo = 0, zero = 0;
    const bool again = fwd_dense_wide_body<KQ, HPC, HALF, MODE, true>(a.g, a.in, a.wd, a.out, a.parts, a.fq, a.kgroups, a.csplit, a.part_stride,
                                                                      (int)blockIdx.x, (int)blockIdx.y, xe, redo, zero, lds);
    if constexpr (WideLds<KQ, HPC, HALF>::TWICE) {
        if (__builtin_expect(!again, 1)) return;
        // (loads the arguments itself: kept for this they take 50 scalar registers more than there are, and vector registers with them)
        typedef const float __attribute__((address_space(1))) *In;
        typedef float __attribute__((address_space(1))) *Out;
        const WideArgs __attribute__((address_space(4))) *p = (const WideArgs __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
        int wg = (int)blockIdx.x, share = (int)blockIdx.y;
        asm volatile("" : "+s"(p), "+s"(wg), "+s"(share));
        Geom g = *(const Geom *)&p->g;
        g.w = (const float *)(In)g.w;
        const FlatGrid fq = *(const FlatGrid *)&p->fq;
        fwd_dense_wide_body<KQ, HPC, HALF, MODE, false>(g, (const float *)(In)p->in, (const float *)(In)p->wd, (float *)(Out)p->out, (float *)(Out)p->parts, fq,
                                                        p->kgroups, p->csplit, p->part_stride, wg, share, xe, redo, zero, lds);
    }
}

}  // namespace
}  // namespace st
