// The dense matrix-core kernel of the unit-stride correlation as a template (FwdDenseCfg, fwd_dense_body,
// fwd_dense_kernel) and the tiling choices of its launches, for the files that instantiate it.
#pragma once
#include "st_common.hpp"
#include "st_split.hpp"

namespace st {
namespace {

// TWD = tile width: 8 (8 rows), 14 (4 rows) or 28 (2 rows); a tile holds at most 64 pixels, i.e.
// two 32-row MFMA blocks; with 14 or 28 columns the last 8 rows of the second block are padding.
//
// MODE selects how tile pixels, taps and input samples relate:
//   0  unit stride: tile pixel (ty,tx), tap (v,u) reads halo pixel (ty+v, tx+u).
//   1  stride 2 (FWD of the stride-2 3x3 layers): halo pixel (2*ty+v, 2*tx+u).
//   2  BWI of a stride-2 3x3 layer with padding 1, one body per parity class (PI,PJ) of the dx
//      positions: the tile is an 8x8 (or 4x14, 2x28) block of the positions (2*i+PI, 2*j+PJ); only
//      the taps whose grid position holds a dy sample contribute (SparseTrain Sec. 3.3): for PI = 0
//      the middle tap reading dy row i, for PI = 1 the outer taps reading dy rows i and i+1; the
//      same along the width.  1, 2, 2 and 4 taps for the four classes instead of 9.
template <int R, int S, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
struct FwdDenseCfg {
    static constexpr int TW = TWD, TH = 64 / TWD, NPIX = TH * TW;
    static constexpr int PSTEP = MODE == 1 ? 2 : 1;                 // halo pixels between neighbouring tile pixels
    static constexpr int NV = MODE == 2 ? (PI ? 2 : 1) : S, NU = MODE == 2 ? (PJ ? 2 : 1) : R, NT = NV * NU;
    static constexpr int HH = MODE == 2 ? TH + PI : (TH - 1) * PSTEP + S;
    static constexpr int HW = MODE == 2 ? TW + PJ : (TW - 1) * PSTEP + R;
    static constexpr int HP = HH * HW;
    // tap t = (kv, ku): halo offset (dv, du) and index of the filter tap in the reformatted copy
    static constexpr int dv(int t) { return t / NU; }
    static constexpr int du(int t) { return t % NU; }
    static constexpr int fv(int t) { return MODE == 2 ? (PI ? 2 * (t / NU) : 1) : t / NU; }
    static constexpr int fu(int t) { return MODE == 2 ? (PJ ? 2 * (t % NU) : 1) : t % NU; }
    static constexpr int ftap(int t) { return fv(t) * R + fu(t); }
    // wavefronts per SIMD the register allocator should aim for: 4, or what the LDS of the
    // workgroups (two halo buffers per pixel tile, 160 KB per compute unit) leaves room for
    static constexpr int minw(int kq)
    {
        const int fit = 163840 / (2 * (4 / kq) * BUF * 4);
        return fit >= 4 ? 4 : (fit >= 1 ? fit : 1);
    }
    // halo buffer: [3 pieces][2 halves of the 16 channels][halo pixel][8 channels] bf16, i.e. 16 bytes per pixel and
    // half, so that neighbouring lanes (pixels) of an operand read are 16 bytes apart
    static constexpr int BUF = ((HP * 24 + 63) / 64) * 64;    // floats per halo buffer
};

// KQ = column blocks (of 32 output channels) per workgroup: 1, 2 or 4; TQ = 4/KQ pixel tiles.
// wg = index of the workgroup among those of the launch, cshare = its share of the channel split;
// lds_base: 2 * TQ halo buffers of BUF floats (fwd_dense_lds_floats), 16-byte aligned.  Every thread of
// the workgroup makes the call (the body contains barriers).
template <int R, int S, int KQ, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
constexpr int fwd_dense_lds_floats() { return 2 * (4 / KQ) * FwdDenseCfg<R, S, TWD, MODE, PI, PJ>::BUF; }

template <int R, int S, int KQ, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
__device__ __forceinline__ void fwd_dense_body(const Geom &g, const float *__restrict__ in, const float *__restrict__ wd,
                                               float *__restrict__ out, float *__restrict__ parts, int tiles_w, int tiles_h, int kgroups,
                                               int total_tiles, int csplit, size_t part_stride, int wg, int cshare,
                                               float *lds_base)
{
    using Cfg = FwdDenseCfg<R, S, TWD, MODE, PI, PJ>;
    constexpr int TH = Cfg::TH, TW = Cfg::TW, HW = Cfg::HW, HP = Cfg::HP, BUF = Cfg::BUF;
    constexpr int TAPS = S * R, TQ = 4 / KQ, NPIX = Cfg::NPIX, NT = Cfg::NT, PSTEP = Cfg::PSTEP;
    constexpr int NLD = (HP * 4 + KQ * 64 - 1) / (KQ * 64);      // float4 loads per lane and block

    // the wavefront index is the same in every lane: kept in a scalar register, and with it every tile coordinate
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int kqi = wave % KQ, tqi = wave / KQ;
    const int kg = wg % kgroups, tg = wg / kgroups;
    const int tile = tg * TQ + tqi;
    const bool tile_ok = tile < total_tiles;
    int t = tile_ok ? tile : 0;
    const int tw = t % tiles_w; t /= tiles_w;
    const int th = t % tiles_h;
    const int n = t / tiles_h;
    const int oh0 = th * TH, ow0 = tw * TW;         // MODE 2: in units of the parity class's own grid
    const int ih0 = MODE == 2 ? oh0 : oh0 * PSTEP - g.ph, iw0 = MODE == 2 ? ow0 : ow0 * PSTEP - g.pw;
    const int CiB = g.Ci / kBlk, KoB = g.Ko / kBlk;
    // channel split (launches with few tiles): share 0 reduces its part of the channel blocks into the output,
    // the others into partial outputs of their own, which sum_partials_kernel adds to it afterwards
    const int cb0 = CiB * cshare / csplit, cb1 = CiB * (cshare + 1) / csplit;
    if (cshare > 0) out = parts + (cshare - 1) * part_stride;
    const int kb32 = kg * KQ + kqi;                 // this wavefront's column block
    const bool k_ok = kb32 * 32 < g.Ko;
    const bool active = tile_ok && k_ok;

    const int l32 = lane % 32, half = lane / 32;

    // running sums of the two pixel blocks, and the matrix cores' own accumulators of the current channel block
    floatx16 acc[2], part[2];
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[pb][r] = 0.f;

    // filter operand: lane supplies the pieces of element (k = kb32*32 + l32, c = half*8 .. half*8+7) from the
    // reformatted copy: 16-byte unit (kb32*CiB*TAPS + step)*192 + piece*64 + lane
    const bf16x8 *bbase = reinterpret_cast<const bf16x8 *>(wd) + (size_t)(k_ok ? kb32 : 0) * CiB * TAPS * 192;
    auto filters = [&](int step, int q) __attribute__((always_inline)) { return bbase[(size_t)step * 192 + q * 64 + lane]; };
    // input operand: lane supplies pixel pb*32 + l32 of the tile, channels half*8 .. half*8+7
    int apix[2];
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
        const int p = min(pb * 32 + l32, NPIX - 1);        // padding rows read a valid pixel; never stored
        apix[pb] = (p / TW) * PSTEP * HW + (p % TW) * PSTEP;
    }

    // halo staging: the KQ wavefronts of a tile split its HP*4 float4 among their KQ*64 lanes
    // (lane index the compiler cannot see through: the addresses are worked out per block instead of being kept in
    // registers across its MFMAs)
    auto load_halo = [&](int cb, float4 (&h)[NLD]) __attribute__((always_inline)) {
        int sl = lane;
        asm volatile("" : "+v"(sl));
        sl += kqi * kWave;
#pragma unroll
        for (int jj = 0; jj < NLD; ++jj) {
            const int idx = jj * (KQ * kWave) + sl;
            const int pix = idx >> 2, q = idx & 3;
            const int a = pix / HW, b = pix % HW;
            const int ih = ih0 + a, iw = iw0 + b;
            h[jj] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (tile_ok && pix < HP && ih >= 0 && ih < g.Hi && iw >= 0 && iw < g.Wi)
                h[jj] = *reinterpret_cast<const float4 *>(in + act_off(n, cb, ih, iw, CiB, g.Hi, g.Wi) + q * 4);
        }
    };
    auto store_halo = [&](float *buf, const float4 (&h)[NLD]) __attribute__((always_inline)) {
        int sl = lane;
        asm volatile("" : "+v"(sl));
        sl += kqi * kWave;
#pragma unroll
        for (int jj = 0; jj < NLD; ++jj) {
            const int idx = jj * (KQ * kWave) + sl;
            const int pix = idx >> 2, q = idx & 3;
            if (pix < HP) {
                bf16x4 p[3];
                split4(h[jj], p);
                bf16x4 *dst = reinterpret_cast<bf16x4 *>(buf) + ((q >> 1) * HP + pix) * 2 + (q & 1);
#pragma unroll
                for (int i = 0; i < 3; ++i) dst[i * (4 * HP)] = p[i];
            }
        }
    };

    float4 hreg[NLD];
    load_halo(cb0, hreg);
    store_halo(lds_base + tqi * BUF, hreg);
    bf16x8 f0 = filters(cb0 * TAPS + Cfg::ftap(0), 0), f1 = filters(cb0 * TAPS + Cfg::ftap(0), 1), f2 = filters(cb0 * TAPS + Cfg::ftap(0), 2);
    __syncthreads();

    for (int cb = cb0; cb < cb1; ++cb) {
        const bf16x8 *lds = reinterpret_cast<const bf16x8 *>(lds_base + (((cb - cb0) & 1) * TQ + tqi) * BUF) + half * HP;
        auto input = [&](int tp, int pb, int q) __attribute__((always_inline)) {
            return lds[apix[pb] + Cfg::dv(tp) * HW + Cfg::du(tp) + q * 2 * HP];
        };
        bf16x8 x0[2], x1[2], x2[2];
#pragma unroll
        for (int pb = 0; pb < 2; ++pb) {
            x0[pb] = input(0, pb, 0);
            x1[pb] = input(0, pb, 1);
            x2[pb] = input(0, pb, 2);
        }
        if (cb + 1 < cb1) load_halo(cb + 1, hreg);          // lands during this block's MFMAs
        // One tap = six products of two pixel blocks.  Every operand register is refilled for the next tap as soon as
        // its last product of this one has been issued (only filter piece 0, used first and last, has a second
        // set), which is what fits the accumulators and both operands into the 128 registers of four wavefronts per
        // SIMD.  The last tap requests the filters of the next block's first one.
        static_for<0, NT>([&](auto T) __attribute__((always_inline)) {
            constexpr int tp = decltype(T)::value;
            constexpr bool last = tp + 1 == NT;
            constexpr int nt = last ? 0 : tp + 1;
            const int nstep = (last ? min(cb + 1, cb1 - 1) : cb) * TAPS + Cfg::ftap(nt);
            auto mul = [&](const bf16x8 &f, const bf16x8 (&x)[2], bool first) __attribute__((always_inline)) {
                if (active) {                               // rows = output channels, columns = pixels
#pragma unroll
                    for (int pb = 0; pb < 2; ++pb)
                        part[pb] = first ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, x[pb], floatx16{}, 0, 0, 0)
                                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, x[pb], part[pb], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            const bf16x8 f0n = filters(nstep, 0);
            mul(f0, x0, tp == 0);
            mul(f2, x0, false);
            f2 = filters(nstep, 2);
            mul(f1, x0, false);
            if constexpr (!last) { x0[0] = input(nt, 0, 0); x0[1] = input(nt, 1, 0); }
            mul(f1, x1, false);
            f1 = filters(nstep, 1);
            mul(f0, x1, false);
            if constexpr (!last) { x1[0] = input(nt, 0, 1); x1[1] = input(nt, 1, 1); }
            mul(f0, x2, false);
            if constexpr (!last) { x2[0] = input(nt, 0, 2); x2[1] = input(nt, 1, 2); }
            f0 = f0n;
        });
        if (active) {
#pragma unroll
            for (int pb = 0; pb < 2; ++pb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[pb][r] = fmaf(cb % 2 ? -1.f : 1.f, part[pb][r], acc[pb][r]);
        }
        if (cb + 1 < cb1) store_halo(lds_base + (((cb + 1 - cb0) & 1) * TQ + tqi) * BUF, hreg);
        __syncthreads();
    }

    // D layout of the 32x32 block: column (pixel) = lane % 32, row (channel) = 8*(r/4) + 4*(lane/32) + r%4:
    // four consecutive channels per group of 4 accumulators, one 16-byte store each
    if (!active) return;
    auto where = [&](int pb, int &oh, int &ow) __attribute__((always_inline)) {
        const int p = pb * 32 + l32;
        oh = MODE == 2 ? 2 * (oh0 + p / TW) + PI : oh0 + p / TW;
        ow = MODE == 2 ? 2 * (ow0 + p % TW) + PJ : ow0 + p % TW;
        return p < NPIX && oh < g.Ho && ow < g.Wo;
    };
    bool finite = true;
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
        int oh, ow;
        if (!where(pb, oh, ow)) continue;
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const int k = kb32 * 32 + 8 * gq + 4 * half;
            if (k >= g.Ko) continue;
            const float4 r = make_float4(acc[pb][4 * gq], acc[pb][4 * gq + 1], acc[pb][4 * gq + 2], acc[pb][4 * gq + 3]);
            finite = finite && split_finite(r.x) && split_finite(r.y) && split_finite(r.z) && split_finite(r.w);
            *reinterpret_cast<float4 *>(out + act_off(n, k / kBlk, oh, ow, KoB, g.Ho, g.Wo) + k % kBlk) = r;
        }
    }
    if (__builtin_expect(!finite, 0)) {             // values outside the range of the bf16 pieces took part
#pragma unroll 1
        for (int i = 0; i < 32; ++i) {
            int oh, ow;
            const int k = kb32 * 32 + 8 * (i % 16 / 4) + 4 * half + i % 4;
            if (!where(i / 16, oh, ow) || k >= g.Ko) continue;
            float *o = out + act_off(n, k / kBlk, oh, ow, KoB, g.Ho, g.Wo) + k % kBlk;
            if (!split_finite(*o)) *o = split_exact_corr(g, in, n, k, oh, ow, cb0, cb1);
        }
    }
}

template <int R, int S, int KQ, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
__global__ __launch_bounds__(256, (FwdDenseCfg<R, S, TWD, MODE, PI, PJ>::minw(KQ))) void fwd_dense_kernel(
    Geom g, const float *__restrict__ in, const float *__restrict__ wd, float *__restrict__ out, float *__restrict__ parts,
    int tiles_w, int tiles_h, int kgroups, int total_tiles, int csplit, size_t part_stride)
{
    if (form_deselected(g.sel, g.want, g.thr)) return;
    __shared__ __attribute__((aligned(16))) float lds_all[fwd_dense_lds_floats<R, S, KQ, TWD, MODE, PI, PJ>()];
    fwd_dense_body<R, S, KQ, TWD, MODE, PI, PJ>(g, in, wd, out, parts, tiles_w, tiles_h, kgroups, total_tiles, csplit, part_stride,
                                                 (int)blockIdx.x, (int)blockIdx.y, lds_all);
}

// Tile width and column blocks per workgroup of a unit-stride launch (the choice launch_rs and
// launch_kq make), and the number of workgroups that results
inline void dense_tiling(const Geom &g, int *twd, int *kq, long long *blocks)
{
    // tile width that divides the row length, if any: 8 -> 8x8, 28 -> 2x28, 14 -> 4x14
    *twd = (g.Wo % 8 != 0 && g.Wo % 28 == 0 && g.Ho % 2 == 0) ? 28
         : (g.Wo % 8 != 0 && g.Wo % 14 == 0 && g.Ho % 4 <= g.Ho % 8) ? 14 : 8;
    *kq = g.Ko > 64 ? 4 : (g.Ko > 32 ? 2 : 1);
    const long long tiles = (long long)ceil_div(g.Wo, *twd) * ceil_div(g.Ho, 64 / *twd) * g.N;
    const int tq = 4 / *kq;
    *blocks = (tiles + tq - 1) / tq * ceil_div(g.Ko, 32 * *kq);
}

// Channel split of the unit-stride 3x3 launches that would leave most of the chip idle (7x7 and 14x14
// layers: a workgroup per pixel tile and 128 output channels gives 128 workgroups for 512 -> 512 @7,
// N = 32, each walking all 512 input channels): up to 8 shares of at least two channel blocks, enough for
// 384 workgroups.  Depends on the geometry only, so that the workspace query and the launch agree.
inline int dense_channel_split(const Geom &g)
{
    if (g.R != 3 || g.S != 3 || g.sw != 1 || g.uw != 1) return 1;
    int twd, kq;
    long long blocks;
    dense_tiling(g, &twd, &kq, &blocks);
    const int CiB = g.Ci / kBlk;
    int cs = 1;
    while (cs < 8 && blocks * cs < 384 && CiB / (cs + 1) >= 2) ++cs;
    return cs;
}

// The partial outputs counted by the workspace query for such a launch (a power of two of them)
inline int dense_channel_split_pow2(const Geom &g)
{
    int twd, kq;
    long long blocks;
    dense_tiling(g, &twd, &kq, &blocks);
    const int CiB = g.Ci / kBlk;
    int cs = 1;
    while (cs < 8 && blocks * cs < 512 && CiB % (cs * 2) == 0 && CiB / (cs * 2) >= 2) cs *= 2;
    return cs;
}

}  // namespace
}  // namespace st
