// Filter-gradient kernels (BWW), unit stride: zero-skipping (vector ALUs) and dense (matrix cores).
//
// Mapping of SparseTrain Sec. 3.4 (Alg. 4-5) onto a CDNA wavefront:
//  * The filter-gradient accumulators are stationary (Sec. 3.4: T gradient vectors stay in
//    registers for the whole sweep): a wavefront owns 64 output channels (one per lane) times
//    8 input channels times R*S taps = 72 registers per lane for a 3x3 filter, which leaves room
//    for 4 wavefronts per SIMD; the scalar work of the zero tests of one wavefront then overlaps
//    the vector work of the others.
//  * The tested operand is the input x.  The tile of x for 64 input channels is staged in LDS by
//    the workgroup (8 wavefronts = 4 channel blocks x 2 halves); with unit stride both tiles are
//    double-buffered and filled by loads that write LDS directly, one tile ahead.  For four pixels at a time one
//    LDS read with a lane per (pixel, channel) followed by one compare and a ballot gives the
//    non-zero mask (the vector compare of Alg. 5, along channels and pixels instead of along the
//    minibatch: the accumulators do not depend on the pixel, so no minibatch transposition of
//    the layout is needed).  Each set bit costs one scalar bit test and branch; the value itself
//    reaches all lanes through a same-address (broadcast) LDS read of the pixel's 8 channels.
//    Which 8 of the 64 channels a wavefront takes is decided per workgroup: the channels with a non-zero in
//    the first tile of its range are dealt round the wavefronts first (whole dead planes would otherwise
//    leave some wavefronts idle at the barrier of every tile).
//  * The other operand, dy at the R*S neighbouring output pixels, is a vector over the lane's
//    output channel read from the LDS halo tile; the 3x6 window of four adjacent pixels is read
//    once per group.
//  * The sum over the minibatch and the image is split over workgroups; each writes a partial
//    gradient to the workspace and a second kernel adds the partials in a fixed order
//    (Sec. 3.4, accumulation of partial results at the end of a sweep), so results are
//    deterministic without floating-point atomics.
#include <cstdio>
#include <atomic>
#include <type_traits>

#include "st_common.hpp"
#include "st_split.hpp"

namespace st {
namespace {

struct BwwArgs {
    int N, C, K, H, W, OH, OW, pw, ph;
    int tiles_w, tiles_h;      // tiles over the input image (sparse) / the output image (dense)
    int units;                 // N * tiles_h * tiles_w
    int splits;                // partial sums; gridDim.x
    int cgroups;               // ceil(C/64)
    // operand selection on the device (st_conv_bww_auto): when sel is set, the launch does nothing
    // unless the sampled zero counts pick the form this launch computes (want: 0 = tests x, 1 = tests dy,
    // 2 = dense; kEitherOperand: a zero-skipping launch that carries the arguments of both of its forms
    // and computes the one selected)
    const unsigned *sel;
    int want;
    // the caller exchanged the operands (dy is the tested one): the tested channels are then the
    // layer's output channels, the lanes its input channels, and the taps come out reversed; the
    // partial sums are still written in the layer's own filter layout
    int swapped;
};

constexpr int kEitherOperand = -1;

// Which of the two argument sets a zero-skipping launch works with.  Returns false when this workgroup
// has nothing to do: the form it computes was not selected, or it lies outside the selected form's grid.
__device__ __forceinline__ bool bww_pick(BwwArgs &A, const BwwArgs &B, const float *&tested, const float *&other)
{
    if (!A.sel) return true;
    const int f = selected_form(A.sel);
    if (A.want != kEitherOperand) return f == A.want;
    if (f == 2) return false;
    if (f == 1) {
        A = B;
        const float *t = tested; tested = other; other = t;
    }
    return (int)blockIdx.x < A.splits && (int)blockIdx.y < ((A.K + 63) / 64) * A.cgroups;
}


// PSTEP = stride of the layer (1 or 2): positions of the halo between neighbouring tile pixels
template <int R, int S, int TH, int TW, int PSTEP = 1>
struct BwwCfg {
    static constexpr int HH = (TH - 1) * PSTEP + S, HW = (TW - 1) * PSTEP + R, HP = HH * HW;
};

// How the pixels of the tested tile, the taps and the pixels of the other operand's halo relate in
// the zero-skipping kernel.  A group is GP = 4 consecutive tested pixels of row a starting at
// column b0; its multiply-adds read a window of the halo that is loaded into registers once.
//   MODE 0  unit stride: pixel j, tap (v,u) <-> window [S-1-v][j+R-1-u]  (window S x (GP+R-1) at (a, b0))
//   MODE 1  stride 2, padding 1, x tested: x pixel (a, b0+j) meets dy row (a+1-v)/2 for the v that make
//           this an integer, the same along the width (window 2 x 3 at (a/2, b0/2); 1, 2 or 4 taps)
//   MODE 2  stride 2, dy tested (operands exchanged by the caller): dy pixel (a, b0+j) meets x pixel
//           (2a+v, 2(b0+j)+u) of its halo for all taps (window 3 x 9 at (2a, 2*b0)); the partial sums
//           are stored with the taps reversed, which is what the exchanged-roles reduction expects
template <int R, int S, int TH, int TW, int MODE>
struct BwwSparseCfg {
    static constexpr int GP = 4;
    static constexpr int HH = MODE == 0 ? TH + S - 1 : MODE == 1 ? TH / 2 + 1 : 2 * (TH - 1) + S;
    static constexpr int HW = MODE == 0 ? TW + R - 1 : MODE == 1 ? TW / 2 + 1 : 2 * (TW - 1) + R;
    static constexpr int HP = HH * HW;
    static constexpr int WR = MODE == 1 ? 2 : S;
    static constexpr int WC = MODE == 0 ? GP + R - 1 : MODE == 1 ? GP / 2 + 1 : 2 * (GP - 1) + R;
    static constexpr int RU = MODE == 1 ? 2 : 1;            // rows whose code differs (row parity)
    static constexpr int wrow0(int a) { return MODE == 0 ? a : MODE == 1 ? a / 2 : 2 * a; }
    static constexpr int wcol0(int b0) { return MODE == 0 ? b0 : MODE == 1 ? b0 / 2 : 2 * b0; }
    static constexpr bool valid(int par, int j, int v, int u)
    {
        return MODE != 1 || (((par + 1 - v) % 2 == 0) && ((j + 1 - u) % 2 == 0));
    }
    static constexpr int wr(int par, int v) { return MODE == 0 ? S - 1 - v : MODE == 1 ? (par + 1 - v) / 2 : v; }
    static constexpr int wc(int j, int u) { return MODE == 0 ? j + R - 1 - u : MODE == 1 ? (j + 1 - u) / 2 : 2 * j + u; }
    static constexpr int slot(int v, int u) { return MODE == 2 ? (S - 1 - v) * R + (R - 1 - u) : v * R + u; }
};

// ------------------------------------------------------------------------------------------
// zero-skipping kernel: tiles run over the INPUT image; LDS holds the x tile (64 channels) and
// the dy halo of the tile (64 output channels)
// ------------------------------------------------------------------------------------------
// x = the tested operand, dy = the other one (the caller exchanges them for the forms that test dy).
// ASYNC (unit stride): both tiles are double-buffered in dynamic LDS (bww_async_lds_bytes) and filled by loads
// that write LDS directly, no registers in between: the tile after the current one is requested right after
// the barrier that opens the current tile's work and lands during it, so no memory round trip is waited for
// and a tile costs one barrier instead of two.
typedef const __attribute__((address_space(1))) void *GlobalPtr;
typedef __attribute__((address_space(3))) void *LdsPtr;
static __device__ __attribute__((aligned(16))) float kZeros16[4] = {0.f, 0.f, 0.f, 0.f};     // source of padding
template <int R, int S, int TH, int TW>
constexpr size_t bww_async_lds_bytes()
{
    using Cfg = BwwSparseCfg<R, S, TH, TW, 0>;
    return (size_t)2 * (Cfg::HP + TH * TW) * 64 * sizeof(float);
}

template <int R, int S, int TH, int TW, int MODE, bool ASYNC = false>
__device__ __forceinline__ void bww_sparse_body(const BwwArgs &A, const float *__restrict__ x, const float *__restrict__ dy,
                                                float *__restrict__ part)
{
    using Cfg = BwwSparseCfg<R, S, TH, TW, MODE>;
    constexpr int HW = Cfg::HW, HP = Cfg::HP, TP = TH * TW;
    constexpr int CH = 8;                 // input channels per wavefront
    constexpr int GP = Cfg::GP;           // pixels per group
    static_assert(TW % GP == 0, "groups must not straddle rows");
    static_assert(TH % Cfg::RU == 0, "row parities come in pairs");
    static_assert(!ASYNC || MODE == 0, "the double-buffered form exists for unit stride only");
    constexpr int WR = Cfg::WR, WC = Cfg::WC;        // dy window of a group
    __shared__ __attribute__((aligned(16))) float dyT_static[ASYNC ? 4 : HP * 64];
    __shared__ __attribute__((aligned(16))) float xT_static[ASYNC ? 4 : TP * 64];
    extern __shared__ __attribute__((aligned(16))) float bww_dynamic_lds[];      // ASYNC: [2][HP + TP][64]
    const float *dyT = dyT_static, *xT = xT_static;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int split = blockIdx.x;
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;
    const int CB = A.C / kBlk, KB = A.K / kBlk;
    const int cbl = wave >> 1, h = wave & 1;          // channel block within the group of 64, half
    const int cb = cg * 4 + cbl;
    const int k = kt * 64 + lane;

    float acc[CH][S * R];
#pragma unroll
    for (int ci = 0; ci < CH; ++ci)
#pragma unroll
        for (int t = 0; t < S * R; ++t) acc[ci][t] = 0.f;

    const int u0 = (int)((long long)A.units * split / A.splits);
    const int u1 = (int)((long long)A.units * (split + 1) / A.splits);

    // ---- which wavefront takes which of the 64 tested channels ----
    // ReLU leaves whole (image, channel) planes dead, and a wavefront's accumulators tie it to its 8 channels
    // for the whole sweep: with the channels handed out in index order a tile takes as long as the wavefront
    // that happens to hold the most alive ones.  The channels that have a non-zero in the first tile of this
    // workgroup's range are therefore dealt round the 8 wavefronts first, the others after them: xT holds
    // channel c at position slot_of[c], and wavefront w works on positions 8w .. 8w+7 as before.  The first
    // tile is a prediction only (a channel that turns out alive later is computed like any other), and every
    // accumulator still sees its pixels in the same order: the results do not depend on the assignment.
    // With exchanged operands the order stays as it is (the 16-byte stores of that epilogue need it).
    __shared__ unsigned alive_w[2];
    __shared__ __attribute__((aligned(16))) unsigned char slot_of[64], chan_of[64];
    if (threadIdx.x < 2) alive_w[threadIdx.x] = 0u;
    __syncthreads();
    if (!A.swapped && u0 < u1) {
        int t = u0;
        const int tw = t % A.tiles_w; t /= A.tiles_w;
        const int th = t % A.tiles_h;
        const int n = t / A.tiles_h;
        unsigned nib = 0u;                                   // a thread's slots all have the same channel quarter
        for (int idx = threadIdx.x; idx < TP * 16; idx += 512) {
            const int pix = idx >> 4, q = idx & 15;
            const int ih = th * TH + pix / TW, iw = tw * TW + pix % TW;
            const int cbq = cg * 4 + (q >> 2);
            if (ih < A.H && iw < A.W && cbq < CB) {
                const float4 val = *reinterpret_cast<const float4 *>(x + act_off(n, cbq, ih, iw, CB, A.H, A.W) + (q & 3) * 4);
                nib |= (val.x != 0.f ? 1u : 0u) | (val.y != 0.f ? 2u : 0u) | (val.z != 0.f ? 4u : 0u) | (val.w != 0.f ? 8u : 0u);
            }
        }
        const int q = threadIdx.x & 15;
        if (nib) atomicOr(&alive_w[q >> 3], nib << ((q & 7) * 4));
    }
    __syncthreads();
    // Loads that write LDS directly put a lane's piece at lane * size: channels in index order, or one 4-byte
    // piece per lane (measured: four times the load instructions cost 5 % of the kernel's time).  The
    // double-buffered form therefore keeps the index order unless at least 8 of the group's channels look dead;
    // then the workgroup stages through registers like the other forms, which can put a value anywhere for free.
    bool dealt = !A.swapped;
    {
        const unsigned long long m = ((unsigned long long)alive_w[1] << 32) | alive_w[0];
        if constexpr (ASYNC) {
            const int real = A.C - cg * 64 < 64 ? A.C - cg * 64 : 64;
            const unsigned long long realmask = real == 64 ? ~0ull : (1ull << real) - 1ull;
            dealt = dealt && __builtin_popcountll(~m & realmask) >= 8;
        }
        if (threadIdx.x < 64) {
            const int c = threadIdx.x;
            const unsigned long long below = (1ull << c) - 1ull;
            const int s = (m >> c) & 1ull ? __builtin_popcountll(m & below)
                                          : __builtin_popcountll(m) + __builtin_popcountll(~m & below);
            const int slot = dealt ? (s & 7) * 8 + (s >> 3) : c;
            slot_of[c] = (unsigned char)slot;
            chan_of[slot] = (unsigned char)c;
        }
    }
    // (the barrier at the top of the tile loop orders these writes before their first use)
    const bool wave_active = A.swapped ? cb < CB : true;

    // ASYNC, channels in index order: request tile `unit` into buffer b, 16 bytes per lane: a wavefront's 64 pieces
    // are 4 pixels of [pixel][64 channels].  Lanes outside the image or beyond the channel count read zeros
    // from kZeros16; lanes beyond the buffer are switched off.  The LDS address of an instruction is the same in
    // every lane (the hardware adds lane * size).
    auto issue = [&](int unit, int b) __attribute__((always_inline)) {
        int t = unit;
        const int tw = t % A.tiles_w; t /= A.tiles_w;
        const int th = t % A.tiles_h;
        const int n = t / A.tiles_h;
        const int ih0 = th * TH, iw0 = tw * TW;
        const int ohs = ih0 + A.ph - (S - 1), ows = iw0 + A.pw - (R - 1);
        float *dst_dy = bww_dynamic_lds + b * ((HP + TP) * 64), *dst_x = dst_dy + HP * 64;
        int ln = lane;
        asm volatile("" : "+v"(ln));                     // (addresses recomputed per tile, not kept in registers)
        constexpr int NI = (HP * 16 + 63) / 64;
        for (int i = wave; i < NI; i += 8) {
            const int idx = i * 64 + ln;
            const int pix = idx >> 4, q = idx & 15;
            const int oh = ohs + pix / HW, ow = ows + pix % HW;
            const int kb = kt * 4 + (q >> 2);
            const float *src = kZeros16;
            if (idx < HP * 16 && oh >= 0 && oh < A.OH && ow >= 0 && ow < A.OW && kb < KB)
                src = dy + act_off(n, kb, oh, ow, KB, A.OH, A.OW) + (q & 3) * 4;
            if (idx < HP * 16)
                __builtin_amdgcn_global_load_lds((GlobalPtr)src, (LdsPtr)(dst_dy + i * 256), 16, 0, 0);
        }
        constexpr int NIX = TP * 16 / 64;
        for (int i = wave; i < NIX; i += 8) {
            const int idx = i * 64 + ln;
            const int pix = idx >> 4, q = idx & 15;
            const int ih = ih0 + pix / TW, iw = iw0 + pix % TW;
            const int cbq = cg * 4 + (q >> 2);
            const float *src = kZeros16;
            if (ih < A.H && iw < A.W && cbq < CB) src = x + act_off(n, cbq, ih, iw, CB, A.H, A.W) + (q & 3) * 4;
            __builtin_amdgcn_global_load_lds((GlobalPtr)src, (LdsPtr)(dst_x + i * 256), 16, 0, 0);
        }
    };
    if constexpr (ASYNC) {
        __syncthreads();                                 // the tables are written
        if (u0 < u1 && !dealt) issue(u0, 0);
    }

    // lane -> (pixel of the group, channel of the block) for the mask read
    const int mpix = lane >> 4, mch = lane & 15;

    for (int unit = u0; unit < u1; ++unit) {
        int t = unit;
        const int tw = t % A.tiles_w; t /= A.tiles_w;
        const int th = t % A.tiles_h;
        const int n = t / A.tiles_h;
        const int ih0 = th * TH, iw0 = tw * TW;
        // first halo pixel of the other operand (MODE 1 assumes padding 1 and even tile origins)
        const int ohs = MODE == 0 ? ih0 + A.ph - (S - 1) : MODE == 1 ? ih0 / 2 : 2 * ih0 - A.ph;
        const int ows = MODE == 0 ? iw0 + A.pw - (R - 1) : MODE == 1 ? iw0 / 2 : 2 * iw0 - A.pw;

        if (ASYNC && !dealt) {
            const int b = (unit - u0) & 1;
            __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wavefront's pieces of the tile have landed
            __syncthreads();                                 // everyone's have; everyone is done with the previous tile
            dyT = bww_dynamic_lds + b * ((HP + TP) * 64);
            xT = dyT + HP * 64;
            if (unit + 1 < u1) issue(unit + 1, b ^ 1);       // lands during this tile's work
        } else {
            // dy[n, kt*64 .. +63, halo] as [pixel][64 k]; x[n, cg*64 .. +63, tile] as [pixel][64 c];
            // 16 float4 per pixel, zeros outside the image and beyond the channel count.  A thread asks for all its
            // 16-byte pieces of the next tile at once, and before the barrier: their round trip overlaps the wait
            // for the wavefronts still at work on the previous tile (one load, one wait, one LDS write at a time,
            // which is what the plain loop compiles to, makes six round trips per tile).
            float *sdst_dy = ASYNC ? bww_dynamic_lds : dyT_static, *sdst_x = ASYNC ? bww_dynamic_lds + HP * 64 : xT_static;
            if constexpr (ASYNC) {
                dyT = sdst_dy;
                xT = sdst_x;
            }
            constexpr int NDY = (HP * 16 + 511) / 512, NX = (TP * 16 + 511) / 512;
            float4 sdy[NDY], sx[NX];
            // (the slot arithmetic is redone for every tile from a thread index the compiler cannot see through:
            // kept across the tile's work as address registers, it spills)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int i = 0; i < NDY; ++i) {
                const int idx = tid + i * 512;
                const int pix = idx >> 4, q = idx & 15;
                const int oh = ohs + pix / HW, ow = ows + pix % HW;
                const int kb = kt * 4 + (q >> 2);
                sdy[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (idx < HP * 16 && oh >= 0 && oh < A.OH && ow >= 0 && ow < A.OW && kb < KB)
                    sdy[i] = *reinterpret_cast<const float4 *>(dy + act_off(n, kb, oh, ow, KB, A.OH, A.OW) + (q & 3) * 4);
            }
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int idx = tid + i * 512;
                const int pix = idx >> 4, q = idx & 15;
                const int ih = ih0 + pix / TW, iw = iw0 + pix % TW;
                const int cbq = cg * 4 + (q >> 2);
                sx[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (idx < TP * 16 && ih < A.H && iw < A.W && cbq < CB)
                    sx[i] = *reinterpret_cast<const float4 *>(x + act_off(n, cbq, ih, iw, CB, A.H, A.W) + (q & 3) * 4);
            }
            __syncthreads();                                     // every wavefront is done with the previous tile
#pragma unroll
            for (int i = 0; i < NDY; ++i) {
                const int idx = tid + i * 512;
                if (idx < HP * 16) *reinterpret_cast<float4 *>(sdst_dy + idx * 4) = sdy[i];       // = [pix][q*4]
            }
            {
                const unsigned sl = reinterpret_cast<const unsigned *>(slot_of)[tid & 15];     // positions of channels 4q .. 4q+3
#pragma unroll
                for (int i = 0; i < NX; ++i) {
                    const int idx = tid + i * 512;
                    const int pix = idx >> 4;
                    if (idx < TP * 16) {
                        sdst_x[pix * 64 + (sl & 0xffu)] = sx[i].x;
                        sdst_x[pix * 64 + ((sl >> 8) & 0xffu)] = sx[i].y;
                        sdst_x[pix * 64 + ((sl >> 16) & 0xffu)] = sx[i].z;
                        sdst_x[pix * 64 + (sl >> 24)] = sx[i].w;
                    }
                }
            }
            __syncthreads();
        }
        if (!wave_active) continue;

        // A multiply-add whose accumulator and two factors all sit in even-numbered or all in odd-numbered
        // registers issues at half rate.  The 8 tested values of a pixel arrive in two aligned groups of four
        // registers, channel ci in one of parity ci % 2; the accumulators of channels 2i + 1 and 2i are handed to
        // the register allocator as (even, odd) pairs here, so that an accumulator never has the parity of
        // its channel's tested value, wherever the window value sits.
        typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int ci = 0; ci < CH; ci += 2)
#pragma unroll
            for (int tp = 0; tp < S * R; ++tp) {
                f2 pr = {acc[ci + 1][tp], acc[ci][tp]};
                asm volatile("" : "+v"(pr));
                acc[ci + 1][tp] = pr.x;
                acc[ci][tp] = pr.y;
            }

        // the mask values of a group are read one group ahead (groups follow each other in memory)
        float mnext = xT[mpix * 64 + cbl * 16 + mch];
        for (int rp = 0; rp < TH / Cfg::RU; ++rp)
        static_for<0, Cfg::RU>([&](auto PAR) __attribute__((always_inline)) {
        constexpr int par = decltype(PAR)::value;            // row parity (MODE 1), else 0
        const int a = rp * Cfg::RU + par;
        for (int b0 = 0; b0 < TW; b0 += GP) {                // groups of GP pixels along the row
            const int g0 = a * TW + b0;
            // non-zero mask of the group: bit 16*j + c for pixel j, channel c of the block
            const float mval = mnext;
            if (g0 + GP < TP) mnext = xT[(g0 + GP + mpix) * 64 + cbl * 16 + mch];
            const unsigned long long m64 = __builtin_amdgcn_ballot_w64(mval != 0.f);
            const unsigned mlo = (unsigned)m64, mhi = (unsigned)(m64 >> 32);
            const unsigned wlo = mlo >> (h * CH), whi = mhi >> (h * CH);     // shifted once per group, not per pixel
            // this wavefront's 8 channels of pixels 0 / 1 (wlo) and 2 / 3 (whi): bits 0-7 and 16-23
            const unsigned any = (wlo | whi) & 0x00FF00FFu;
            if (any == 0u) continue;                         // nothing to do for these 4 pixels x 8 channels
            // window of the other operand's halo, this lane's channel
            float dyw[WR][WC];
            const int w0 = Cfg::wrow0(a) * HW + Cfg::wcol0(b0);
#pragma unroll
            for (int r = 0; r < WR; ++r)
#pragma unroll
                for (int cc = 0; cc < WC; ++cc) dyw[r][cc] = dyT[(w0 + r * HW + cc) * 64 + lane];
            // x of pixel 0 of the group: 8 channels, same address in all lanes
            const float4 *xq = reinterpret_cast<const float4 *>(xT + g0 * 64 + cbl * 16 + h * CH);
            float4 xlo = xq[0], xhi = xq[1];
            __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): window and first pixel are here
            static_for<0, GP>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = decltype(J)::value;
                float4 nlo = xlo, nhi = xhi;
                if constexpr (j + 1 < GP) {                  // next pixel's values fly during this pixel's work
                    nlo = xq[(j + 1) * 16];
                    nhi = xq[(j + 1) * 16 + 1];
                }
                const float xs[CH] = {xlo.x, xlo.y, xlo.z, xlo.w, xhi.x, xhi.y, xhi.z, xhi.w};
                // this wavefront's 8 channels of pixel j sit at constant bit positions of the shifted mask words
                const unsigned mw = (j < 2) ? wlo : whi;
                constexpr int sh = (j % 2) * 16;
                if (__builtin_expect((mw & (0xFFu << sh)) != 0u, 1)) {
                    static_for<0, CH>([&](auto CI) __attribute__((always_inline)) {
                        constexpr int ci = decltype(CI)::value;
                        if (__builtin_expect((mw & (1u << (sh + ci))) != 0u, 1)) {
#pragma unroll
                            for (int v = 0; v < S; ++v)
#pragma unroll
                                for (int u = 0; u < R; ++u)
                                    if (Cfg::valid(par, j, v, u))
                                        acc[ci][Cfg::slot(v, u)] = fmaf(xs[ci], dyw[Cfg::wr(par, v)][Cfg::wc(j, u)],
                                                                        acc[ci][Cfg::slot(v, u)]);
                        }
                    });
                }
                if constexpr (j + 1 < GP) __builtin_amdgcn_s_waitcnt(0xC07F);
                xlo = nlo;
                xhi = nhi;
            });
        }
        });
    }

    if (wave_active && k < A.K) {
        const int kb = k / kBlk, ki = k % kBlk;
        float *pbase = part + (size_t)split * A.K * A.C * (S * R);
        if (!A.swapped) {
#pragma unroll
            for (int ci = 0; ci < CH; ++ci) {
                const int c = cg * 64 + chan_of[wave * CH + ci];        // the channel this accumulator row belongs to
                if (c >= A.C) continue;
                float *p = pbase + ((size_t)kb * CB + c / kBlk) * (S * R * kBlk * kBlk) + (c % kBlk) * kBlk + ki;
#pragma unroll
                for (int tp = 0; tp < S * R; ++tp) p[tp * (kBlk * kBlk)] = acc[ci][tp];
            }
        } else {
            // layer's block [cb: its output channels][kb: its input channels], element [ki][h*8 + ci]: the
            // lane's 8 tested channels are consecutive, the taps are reversed
            // The values pass through an OR with a zero the compiler cannot see, i.e. through fresh registers:
            // handed to the 16-byte stores directly, the accumulators would have to sit in aligned groups of
            // four, and that numbering makes the multiply-adds of the main loop 6 % slower (measured), for the
            // x-testing form as well since it is the same code.
            const unsigned zero = (unsigned)(A.swapped - 1);
            auto fresh = [&](float v) __attribute__((always_inline)) { return __uint_as_float(__float_as_uint(v) | zero); };
            float *p = pbase + ((size_t)cb * KB + kb) * (S * R * kBlk * kBlk) + ki * kBlk + h * CH;
#pragma unroll
            for (int tp = 0; tp < S * R; ++tp) {
                float4 *q = reinterpret_cast<float4 *>(p + (S * R - 1 - tp) * (kBlk * kBlk));
                q[0] = make_float4(fresh(acc[0][tp]), fresh(acc[1][tp]), fresh(acc[2][tp]), fresh(acc[3][tp]));
                q[1] = make_float4(fresh(acc[4][tp]), fresh(acc[5][tp]), fresh(acc[6][tp]), fresh(acc[7][tp]));
            }
        }
    }
}

template <int R, int S, int TH, int TW, int MODE = 0>
__global__ __launch_bounds__(512, 4) void bww_sparse_kernel(BwwArgs A, const float *__restrict__ x,
                                                            const float *__restrict__ dy, float *__restrict__ part)
{
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    bww_sparse_body<R, S, TH, TW, MODE, MODE == 0>(A, x, dy, part);
}

// st_conv_bww_auto: one launch for both zero-skipping forms of a unit-stride layer.  It carries the arguments of
// the x-testing form (A) and of the dy-testing form (B, operands exchanged) and computes the one the sampled
// counts select; a kernel of its own, so that the kernel of the direct calls keeps its code (with the choice
// inside, that one ran 6 % slower).
template <int R, int S, int TH, int TW>
__global__ __launch_bounds__(512, 4) void bww_sparse_either_kernel(BwwArgs A, BwwArgs B, const float *x, const float *dy,
                                                                   float *__restrict__ part)
{
    const float *tested = x, *other = dy;
    if (!bww_pick(A, B, tested, other)) return;         // uniform over the workgroup, before any barrier
    bww_sparse_body<R, S, TH, TW, 0, true>(A, tested, other, part);
}

// ------------------------------------------------------------------------------------------
// dense kernels: tiles run over the OUTPUT image; LDS holds the dy tile and the x halo as bf16 pieces (st_split.hpp), six
// products per filter tap.  The reduction runs over thousands of pixels: the products of a tile are added up in a fresh accumulator
// and joined to the tap's fp32 sum on the vector ALUs, so a sum takes one rounding per tile (3136 terms: error 2e-7 of the norm;
// 7e-7 with v_mfma_f32_32x32x2_f32, 8e-7 with the matrix cores' own long sums).
//
// Small tiles: 144 sums, short accumulators, the operands of a tap and the next tile's loads then fit the 256 registers of two
// wavefronts per SIMD, and two workgroups share a compute unit, so that one's staging meets the other's arithmetic.
//
// Stride 2: tiles of 2 x 8 pixels, one v_mfma_f32_32x32x16_bf16 (rows = 32 output channels, columns = 32 input channels, reduction =
// the 16 pixels) per product, two barriers per 54 of them of a wavefront.  128->128 @56, N = 32, 82 us (98 with
// v_mfma_f32_32x32x2_f32 on 98-pixel tiles).  Unit stride: see the kernel after it.
// ------------------------------------------------------------------------------------------
template <int R, int S, int TH, int TW, int PSTEP>
struct BwwDenseCfg {
    using Halo = BwwCfg<R, S, TH, TW, PSTEP>;
    static constexpr int TP = TH * TW, P = (TP + 15) / 16 * 16;         // tile pixels, padded to whole 16s
    // [piece][half of the 64 channels][pixel][32 channels], 64 bytes a pixel
    static constexpr int XB = Halo::HP * 64, DB = P * 64;
    static constexpr int LDS = 6 * (XB + DB);
};

// Staging of both dense kernels.  A thread's 16-byte pieces of a tile (dy tile, then x halo: 16 float4 per pixel, zeros outside the
// image and beyond the channel count) are asked for while the previous tile is being multiplied, split and written to LDS after
// it: the memory round trip is hidden behind the matrix work.
template <int R, int S, int TH, int TW, int PSTEP>
struct BwwDenseStage {
    using Cfg = BwwDenseCfg<R, S, TH, TW, PSTEP>;
    static constexpr int HW = Cfg::Halo::HW, HP = Cfg::Halo::HP, ND = (Cfg::P * 16 + 255) / 256, NXH = (HP * 16 + 255) / 256;
    float4 sd[ND], sx[NXH];

    // Every other tile is added up with the opposite sign (its dy negated, its sum subtracted): what the matrix cores cut off
    // leaves a small bias, which over 10^5 pixels would outgrow the rounding errors (256->256 @56, N = 32: error 7.8e-7 of the
    // norm with one sign, 2.7e-7 with both).
    static __device__ __forceinline__ float sign(int unit) { return unit % 2 ? -1.f : 1.f; }

    __device__ __forceinline__ void fetch(const BwwArgs &A, const float *__restrict__ x, const float *__restrict__ dy, int kt, int cg, int unit)
    {
        int t = unit;
        const int tw = t % A.tiles_w; t /= A.tiles_w;
        const int th = t % A.tiles_h;
        const int n = t / A.tiles_h;
        const int CB = A.C / kBlk, KB = A.K / kBlk;
        const int oh0 = th * TH, ow0 = tw * TW, ih0 = oh0 * PSTEP - A.ph, iw0 = ow0 * PSTEP - A.pw;
        // (thread index the compiler cannot see through: the slot arithmetic is redone per tile instead of
        // being kept in address registers across the tile's work)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int idx = tid + i * 256;
            const int pix = idx >> 4, q = idx & 15;
            const int oh = oh0 + pix / TW, ow = ow0 + pix % TW;
            const int kb = kt * 4 + (q >> 2);
            sd[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (pix < Cfg::TP && oh < A.OH && ow < A.OW && kb < KB)
                sd[i] = *reinterpret_cast<const float4 *>(dy + act_off(n, kb, oh, ow, KB, A.OH, A.OW) + (q & 3) * 4);
        }
#pragma unroll
        for (int i = 0; i < NXH; ++i) {
            const int idx = tid + i * 256;
            const int pix = idx >> 4, q = idx & 15;
            const int ih = ih0 + pix / HW, iw = iw0 + pix % HW;
            const int cb = cg * 4 + (q >> 2);
            sx[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (pix < HP && ih >= 0 && ih < A.H && iw >= 0 && iw < A.W && cb < CB)
                sx[i] = *reinterpret_cast<const float4 *>(x + act_off(n, cb, ih, iw, CB, A.H, A.W) + (q & 3) * 4);
        }
    }

    // into buf: the pieces of the dy tile, then those of the halo
    __device__ __forceinline__ void stash(int unit, char *buf) const
    {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int i = 0; i < ND + NXH; ++i) {
            const bool isx = i >= ND;
            const int idx = tid + (isx ? i - ND : i) * 256, pix = idx >> 4, q = idx & 15, bytes = isx ? Cfg::XB : Cfg::DB;
            if (pix >= (isx ? HP : Cfg::P)) continue;
            bf16x4 p[3];
            split4(isx ? sx[isx ? i - ND : 0] : sd[isx ? 0 : i], isx ? kSplitScale : sign(unit) * kSplitScale, p);
            char *dst = buf + (isx ? 6 * Cfg::DB : 0) + (q >> 3) * bytes + pix * 64 + (q & 7) * 8;
#pragma unroll
            for (int j = 0; j < 3; ++j) *reinterpret_cast<bf16x4 *>(dst + j * 2 * bytes) = p[j];
        }
    }
};

// The 32 x 32 block (output channels k32 .., input channels c32 ..) of a partial gradient once more with fp32 multiply-adds
// on the matrix cores, operands straight from memory: tiles u0 .. u1-1, all taps.  A sample outside the image takes its
// dy factor out with it (0 * inf would be NaN).  The 64 lanes of a wavefront make the call together.
// 256->256 @56, N = 8, us: 170 for ordinary values, one infinity 563, everywhere 607 (element by element, each by one lane, one
// infinity or subnormal took 27000).
template <int R, int S, int TH, int TW, int PSTEP>
__device__ __forceinline__ void bww_redo(const BwwArgs &A, const float *x, const float *dy, int k32, int c32, int u0, int u1, floatx16 (&acc)[S * R])
{
    static_assert(TH * TW % 2 == 0, "an instruction takes two pixels");
    const int lane = threadIdx.x % kWave, l32 = lane % 32, half = lane / 32;
    const int k = min(k32 + l32, A.K - 1), c = min(c32 + l32, A.C - 1);        // (rows and columns past the end are not stored)
#pragma unroll
    for (int t = 0; t < S * R; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll 1
    for (int unit = u0; unit < u1; ++unit) {
        int t = unit;
        const int tw = t % A.tiles_w; t /= A.tiles_w;
        const int th = t % A.tiles_h, n = t / A.tiles_h;
        const float *xc = x + act_off(n, c / kBlk, 0, 0, A.C / kBlk, A.H, A.W) + c % kBlk;
        const float *dk = dy + act_off(n, k / kBlk, 0, 0, A.K / kBlk, A.OH, A.OW) + k % kBlk;
#pragma unroll 2
        for (int pp = 0; pp < TH * TW / 2; ++pp) {
            const int p = 2 * pp + half, oh = th * TH + p / TW, ow = tw * TW + p % TW;
            const bool in = oh < A.OH && ow < A.OW;
            const float d = dk[in ? (oh * A.OW + ow) * kBlk : 0];
            float xv[S * R];
            bool meets[S * R];
#pragma unroll
            for (int tap = 0; tap < S * R; ++tap) {
                const int ih = oh * PSTEP - A.ph + tap / R, iw = ow * PSTEP - A.pw + tap % R;
                meets[tap] = in && ih >= 0 && ih < A.H && iw >= 0 && iw < A.W;
                xv[tap] = xc[meets[tap] ? (ih * A.W + iw) * kBlk : 0];
            }
#pragma unroll
            for (int tap = 0; tap < S * R; ++tap)
                acc[tap] = __builtin_amdgcn_mfma_f32_32x32x2f32(meets[tap] ? d : 0.f, meets[tap] ? xv[tap] : 0.f, acc[tap], 0, 0, 0);
        }
    }
}

// SHORT: for workgroups of few tiles, see the products below.
template <int R, int S, int TH, int TW, int PSTEP, bool SHORT>
__global__ __launch_bounds__(256, 2) void bww_dense_kernel(BwwArgs A, const float *__restrict__ x,
                                                           const float *__restrict__ dy, float *__restrict__ part)
{
    using Cfg = BwwDenseCfg<R, S, TH, TW, PSTEP>;
    using Stage = BwwDenseStage<R, S, TH, TW, PSTEP>;
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    constexpr int HW = Cfg::Halo::HW, XB = Cfg::XB, DB = Cfg::DB;
    static_assert(Cfg::TP == 16, "a tile is the reduction of one instruction");
    __shared__ __attribute__((aligned(16))) char lds[Cfg::LDS];

    // the wavefront index is the same in every lane: kept in a scalar register, and with it every tile coordinate
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l32 = lane % 32, half = lane / 32;
    const int kh = wave % 2, ch = wave / 2;
    const int split = blockIdx.x;
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;
    const int CB = A.C / kBlk;
    const bool active = kt * 64 + kh * 32 < A.K && cg * 64 + ch * 32 < A.C;

    floatx16 acc[S * R];
#pragma unroll
    for (int t = 0; t < S * R; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

    const int u0 = (int)((long long)A.units * split / A.splits);
    const int u1 = (int)((long long)A.units * (split + 1) / A.splits);

    // this lane's addresses: pixel half*8 + i*4 + (lane % 16) / 4 of the tile for read i
    LdsTr dp, xp[2];
    {
        const int px = half * 8 + lane % 16 / 4;
        dp = (LdsTr)(lds + kh * DB + px * 64 + split_tr_lane(lane));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int p = i * 4 + px;
            xp[i] = (LdsTr)(lds + 6 * DB + ch * XB + (p / TW * HW + p % TW) * (PSTEP * 64) + split_tr_lane(lane));
        }
    }

    Stage stage;
    if (u0 < u1) stage.fetch(A, x, dy, kt, cg, u0);
    for (int unit = u0; unit < u1; ++unit) {
        __syncthreads();                                     // every wavefront is done with the previous tile
        stage.stash(unit, lds);
        __syncthreads();
        if (unit + 1 < u1) stage.fetch(A, x, dy, kt, cg, unit + 1);          // in flight during this tile's MFMAs
        if (!active) continue;

        bf16x8 d[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) d[q] = split_tr_read(dp + q * 2 * DB / 8, dp + (q * 2 * DB + 256) / 8);
        auto input = [&](int tap, bf16x8 (&f)[3]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int off = (q * 2 * XB + (tap / R * HW + tap % R) * 64) / 8;
                f[q] = split_tr_read(xp[0] + off, xp[1] + off);
            }
        };
        bf16x8 f[3];
        input(0, f);
        static_for<0, S * R>([&](auto T) __attribute__((always_inline)) {
            constexpr int tap = decltype(T)::value;
            bf16x8 fn[3];
            if constexpr (tap + 1 < S * R) input(tap + 1, fn);
            __builtin_amdgcn_sched_barrier(0);              // the next tap's reads go ahead of this tap's products
            floatx16 t = {};
            if constexpr (SHORT) {                          // two of the products usually left out
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[2], f[1], t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[1], f[2], t, 0, 0, 0);
            }
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[2], f[0], t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[0], f[2], t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[1], f[1], t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[1], f[0], t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[0], f[1], t, 0, 0, 0);
            // The products of the leading pieces on top of the others cut the others off at their own last bit.  Beside the
            // rounding of a sum over many steps that is nothing; in a launch of few tiles the two meet in an fp32 addition
            // instead, and two more of the small products are formed (SHORT).  (16 to 162 pixels with 4 % non-zero
            // products: 1.13-1.34 -> 1.00-1.04 times the fp32 instruction's error; it takes 5 % longer on long sums, whose
            // error it does not change.)
            if constexpr (SHORT) {
                const floatx16 h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[0], f[0], floatx16{}, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r) t[r] += h[r];
            } else {
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[0], f[0], t, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tap][r] = unit % 2 ? acc[tap][r] - t[r] : acc[tap][r] + t[r];
            if constexpr (tap + 1 < S * R) {
#pragma unroll
                for (int q = 0; q < 3; ++q) f[q] = fn[q];
            }
        });
    }
    if (!active) return;

    // D layout of the 32x32 block: column (c) = lane % 32, row (k) = 8*(r/4) + 4*(lane/32) + r%4: four consecutive output
    // channels per group of 4 accumulators, one 16-byte store each
    const int k32 = kt * 64 + kh * 32, c32 = cg * 64 + ch * 32, c = c32 + l32;
    float *pbase = part + (size_t)split * A.K * A.C * (S * R);
    auto element = [&](int k, int tap) __attribute__((always_inline)) {
        return pbase + (((size_t)(k / kBlk) * CB + c / kBlk) * (S * R) + tap) * (kBlk * kBlk) + (c % kBlk) * kBlk + k % kBlk;
    };
    bool finite = true;
    if (c < A.C) {
#pragma unroll
        for (int tap = 0; tap < S * R; ++tap)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const int k = k32 + 8 * gq + 4 * half;
                if (k >= A.K) continue;
                const float4 v = make_float4(acc[tap][4 * gq] * kSplitUnscale, acc[tap][4 * gq + 1] * kSplitUnscale,
                                             acc[tap][4 * gq + 2] * kSplitUnscale, acc[tap][4 * gq + 3] * kSplitUnscale);
                finite = finite && split_finite(v);
                *reinterpret_cast<float4 *>(element(k, tap)) = v;
            }
    }
    // sums that values outside the range of the scaled pieces took part in
    if (__builtin_expect(__ballot(!finite) != 0, 0)) {
        bww_redo<R, S, TH, TW, PSTEP>(A, x, dy, k32, c32, u0, u1, acc);
        if (c >= A.C) return;
#pragma unroll
        for (int tap = 0; tap < S * R; ++tap)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k32 + 8 * (r / 4) + 4 * half + r % 4;
                if (k < A.K && !split_finite(*element(k, tap))) *element(k, tap) = acc[tap][r];
            }
    }
}

// Staging of the unit-stride kernel: as above, with the vector instructions that cost the matrix cores their issue slots taken out (203 -> 92 to ask for a
// tile, 191 -> 167 to split and write it: 256->256 @56, N = 32, 494 -> 478 us, 512->512 @28 547 -> 529, 64->64 @224 536 -> 518).  Addresses are 32 bits behind a buffer descriptor per image, whose range check returns the zeros of channels past
// the end; pixels outside the image ask beyond it.  A row and a column are compared as one packed pair.  Layout of a buffer: [pieces][2 halves of the 64
// channels][32 pixels][32 channels] of dy, the same of x with XPX pixels.
constexpr int kBwwNoTileRow = 40000;            // row of tiles that do not exist: images of these sizes have fewer (bww_big_image)
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Bytes of sample (h, w) within a channel block.  Unsigned: above and left of the image it wraps, as the sums it takes part in do, and for the rows of tiles
// that do not exist, whose offset no one uses, it may
constexpr unsigned bww_sample_offset(int h, int w, int W) { return ((unsigned)h * (unsigned)W + (unsigned)w) * (unsigned)(kBlk * 4); }
static_assert(bww_sample_offset(kBwwNoTileRow, 31999, 32000) != 0 && bww_sample_offset(-1, -1, 5) + 6u * (kBlk * 4) == 0, "(an overflow of int is no constant)");
// BIG: images of any size (bww_big_image), with 64-bit addresses.
template <int TH, int TW, bool BIG = false>
struct BwwWideStage {
    static constexpr int HW = TW + 2, HP = (TH + 2) * HW, XPX = 64, DPX = 32;       // (halos of 60 and 64 samples)
    static constexpr int XB = XPX * 64, DB = DPX * 64;
    static_assert(HP <= XPX && HP > XPX - 16 && TH * TW <= DPX && TH * TW > DPX - 16, "whole rounds of 256 threads");
    static constexpr int bytes(int pieces) { return pieces * 2 * (XB + DB); }
    struct Tile {
        int n, th, tw;
        __device__ __forceinline__ void start(const BwwArgs &A, int unit)
        {
            tw = unit % A.tiles_w;
            th = unit / A.tiles_w % A.tiles_h;
            n = unit / A.tiles_w / A.tiles_h;
        }
        __device__ __forceinline__ void step(const BwwArgs &A)
        {
            if (++tw == A.tiles_w) {
                tw = 0;
                if (++th == A.tiles_h) { th = 0; ++n; }
            }
        }
    };

    // 16-byte pieces of channel blocks cb .. cb+3 of image n of a tensor (CB blocks of H x W): a block of samples of COLS columns whose first one is
    // (h0, w0); PX of them, zeros for those outside the image
    template <int COLS, int PX, int NP>
    static __device__ __forceinline__ void ask(const float *t, int n, int cb, int CB, int h0, int w0, int H, int W, float4 (&to)[NP])
    {
        // (thread index the compiler cannot see through: see above)
        int tid = threadIdx.x % 256;
        asm volatile("" : "+v"(tid));
        const int q = tid & 15, pix0 = tid >> 4;
        const float *base = t + ((size_t)n * CB + cb) * H * W * kBlk;
        if constexpr (BIG) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int pix = pix0 + i * 16, h = h0 + pix / COLS, w = w0 + pix % COLS;
                to[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (pix < PX && h >= 0 && h < H && w >= 0 && w < W && cb + (q >> 2) < CB)
                    to[i] = *reinterpret_cast<const float4 *>(base + ((size_t)(q >> 2) * H * W + (size_t)h * W + w) * kBlk + (q & 3) * 4);
            }
        } else {
            const __amdgpu_buffer_rsrc_t from =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, min(4, CB - cb) * (H * W) * (kBlk * 4), 0x00020000);
            const unsigned at = bww_sample_offset(h0, w0, W) + (unsigned)((q >> 2) * (H * W * (kBlk * 4)) + (q & 3) * 16);
            const u16x2 first = {(unsigned short)h0, (unsigned short)w0}, last = {(unsigned short)(H - 1), (unsigned short)(W - 1)};
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const unsigned pix = pix0 + i * 16, r = pix / COLS, c = pix % COLS;
                const u16x2 hw = __builtin_bit_cast(u16x2, r | c << 16) + first, in = __builtin_elementwise_min(hw, last);
                const bool ok = __builtin_bit_cast(unsigned, in) == __builtin_bit_cast(unsigned, hw) && ((i + 1) * 16 <= PX || (int)pix < PX);
                const unsigned off = ok ? at + r * (W * (kBlk * 4)) + c * (kBlk * 4) : 0x80000000u;
                to[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(from, (int)off, 0, 0));
            }
        }
    }
    static __device__ __forceinline__ void fetch_dy(const BwwArgs &A, const float *__restrict__ dy, int kt, const Tile &t, float4 (&sd)[2])
    {
        ask<TW, TH * TW>(dy, t.n, kt * 4, A.K / kBlk, t.th * TH, t.tw * TW, A.OH, A.OW, sd);
    }
    static __device__ __forceinline__ void fetch_x(const BwwArgs &A, const float *__restrict__ x, int cg, const Tile &t, float4 (&sx)[4])
    {
        ask<HW, HP>(x, t.n, cg * 4, A.C / kBlk, t.th * TH - A.ph, t.tw * TW - A.pw, A.H, A.W, sx);
    }
    // three bf16 pieces of a tile
    static __device__ __forceinline__ void stash(const float4 (&sd)[2], const float4 (&sx)[4], float sign, char *buf)
    {
        int tid = threadIdx.x % 256;
        asm volatile("" : "+v"(tid));
        const int q = tid & 15, pix0 = tid >> 4, at = pix0 * 64 + (q & 7) * 8;
        char *d = buf + (q >> 3) * DB + at, *h = buf + 6 * DB + (q >> 3) * XB + at;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            bf16x4 p[3];
            split4(i < 2 ? sd[i < 2 ? i : 0] : sx[i < 2 ? 0 : i - 2], i < 2 ? sign * kSplitScale : kSplitScale, p);
#pragma unroll
            for (int j = 0; j < 3; ++j) *reinterpret_cast<bf16x4 *>(i < 2 ? d + i * 1024 + j * 2 * DB : h + (i - 2) * 1024 + j * 2 * XB) = p[j];
        }
    }
    // two f16 pieces of one operand's part of a tile (halves of the channels BYTES apart), scale sign 2^e; returns how many of its fours hold a value
    // below the pieces' range
    template <int BYTES, int NP>
    static __device__ __forceinline__ unsigned stash_half(const float4 (&v)[NP], float sign, int e, char *buf)
    {
        int tid = threadIdx.x % 256;
        asm volatile("" : "+v"(tid));
        const int q = tid & 15, pix0 = tid >> 4;
        char *d = buf + (q >> 3) * BYTES + pix0 * 64 + (q & 7) * 8;
        const float scale = sign * half_scale(e), low = sign * half_scale(e + 11);
        unsigned lows = 0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            f16x4 p[2];
            half4(v[i], scale, low, p);
            lows += half_low(v[i], half_low_key(e));
#pragma unroll
            for (int j = 0; j < 2; ++j) *reinterpret_cast<f16x4 *>(d + i * 1024 + j * 2 * BYTES) = p[j];
            __builtin_amdgcn_sched_barrier(0);                  // a piece at a time: there are no registers for several
        }
        return lows;
    }
};

// A workgroup of the unit-stride kernel on bf16 pieces is one team of four wavefronts or (bww_teams) two, which take tiles of
// their own and add their sums up in LDS: what used to be two workgroups on a compute unit writes one set of partial gradients instead of two, and the
// final sum reads half as many: 32 x 128->128 @28 59.5 -> 56.0 us.
// Tiles of the teams: first, then one past the last of each, steps = the most tiles of one of them.
template <int TEAMS>
struct BwwTeam {
    int team, first, u0, u1, last, steps;
    __device__ __forceinline__ BwwTeam(const BwwArgs &A)
    {
        team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
        auto bound = [&](int i) __attribute__((always_inline)) {
            return (int)((long long)A.units * min((int)blockIdx.x * TEAMS + i, A.splits) / A.splits);
        };
        first = bound(0);
        last = bound(TEAMS);
        u0 = bound(team);
        u1 = bound(team + 1);
        steps = TEAMS == 1 ? u1 - u0 : max(bound(1) - first, last - bound(1));
    }
    // the sums of both in those of the first; every thread makes the call.  False: nothing left to do
    template <int N>
    __device__ __forceinline__ bool join(floatx4 (&acc)[N][2][2], bool active, int wave, int lane, char *lds) const
    {
        if constexpr (TEAMS == 1) return active;
        __syncthreads();                                        // every wavefront is done with its tiles
        floatx4 *ex = reinterpret_cast<floatx4 *>(lds) + wave * (N * 4 * kWave) + lane;
        if (team == 1 && active) {
#pragma unroll
            for (int t = 0; t < N * 4; ++t) ex[t * kWave] = acc[t / 4][t / 2 % 2][t % 2];
        }
        __syncthreads();
        if (team == 1 || !active) return false;
#pragma unroll
        for (int t = 0; t < N * 4; ++t) acc[t / 4][t / 2 % 2][t % 2] += ex[t * kWave];
        return true;
    }
};

// The same for unit stride (the kernel above serves stride 2) with v_mfma_f32_16x16x32_bf16, 32 pixels (a whole tile) at a
// time: it reaches 2050 TFLOP/s where 32x32x16 reaches 1760 (st_fwd_dense_wide.hpp), and its sum joins the running one once per
// tile instead of once per 16 pixels.  A wavefront's 32 x 32 channels are 2 x 2 blocks of 16 x 16.  The registers are full (144 sums,
// 16 of a tap, 48 operands, 24 of the next tile), so every x operand is read again for the next tap as soon as its last product
// has been issued.  N = 32, us, 32x32x16 -> now (both with the final sum): 256->256 @56 554 -> 490 (242 TFLOP/s), 512->512 @28
// 607 -> 542, @14 170 -> 154, 64->64 @224 614 -> 540, 128->128 @28 63.5 -> 61.6, one image 64->64 @14 14.4 -> 12.5; error against
// 64 bits 2.55e-7 -> 1.86e-7, 2.72e-7 -> 2.03e-7, 1.46e-7 -> 1.15e-7, 2.62e-7 -> 1.95e-7, 9.3e-8 -> 8.2e-8, 4.5e-8 -> 3.8e-8.
// Bound: power (see there) and, beside the products, splitting and stashing the next tile.
// lds_all: for each team two buffers of three pieces, which take turns
template <int R, int S, int TH, int TW, bool SHORT, bool BIG, int TEAMS>
__device__ __forceinline__ void bww_dense_wide_body(const BwwArgs &A, const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, char *lds_all)
{
    using Stage = BwwWideStage<TH, TW, BIG>;
    constexpr int HW = Stage::HW, TP = TH * TW, XB = Stage::XB, DB = Stage::DB;

    // the wavefront index is the same in every lane: kept in a scalar register, and with it every tile coordinate
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x % 256 / kWave), lane = threadIdx.x % kWave;
    const int l16 = lane % 16, grp = lane / 16;
    const int kh = wave % 2, ch = wave / 2;
    const BwwTeam<TEAMS> team(A);
    const int u0 = team.u0, u1 = team.u1;
    char *const lds = lds_all + team.team * (2 * Stage::bytes(3));
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;
    const int CB = A.C / kBlk;
    const bool active = kt * 64 + kh * 32 < A.K && cg * 64 + ch * 32 < A.C;

    floatx4 acc[S * R][2][2];                           // [tap][16 k][16 c]
#pragma unroll
    for (int t = 0; t < S * R; ++t)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[t][kb][cb] = floatx4{0.f, 0.f, 0.f, 0.f};

    // the next tile is written into the other buffer: one barrier a tile (256->256 @56 502 -> 490; a piece after each of the last taps
    // has no registers, 76 spilled, 514)
    typename Stage::Tile next;
    next.start(A, u0);
    float4 sd[2], sx[4];
    auto fetch = [&]() __attribute__((always_inline)) {
        Stage::fetch_dy(A, dy, kt, next, sd);
        Stage::fetch_x(A, x, cg, next, sx);
        next.step(A);
    };
    auto sign = [](int unit) __attribute__((always_inline)) { return unit % 2 ? -1.f : 1.f; };        // (BwwDenseStage)

    // operands: lane l takes channel l % 16 of a block and pixels 8*(l/16) .. +7 of the tile, four per transposing read, for which
    // it supplies the address of 8 bytes of pixel (l % 16) / 4 of the four
    int dp, xp[2];
    {
        const int px = grp * 8 + l16 / 4, chan = l16 % 4 * 8;
        dp = kh * DB + px * 64 + chan;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int p = min(px + i * 4, TP - 1);              // (the padding's dy is zero)
            xp[i] = 6 * DB + ch * XB + (p / TW * HW + p % TW) * 64 + chan;
        }
    }

    if (TEAMS == 1 || u0 < u1) {                             // (one team has at least one tile)
        fetch();
        Stage::stash(sd, sx, sign(u0), lds);
    }
    __syncthreads();
    for (int unit = u0; unit < u1; ++unit) {
        char *const buf = lds + (unit - u0) % 2 * Stage::bytes(3);
        if (unit + 1 < u1) fetch();                          // in flight during this tile's MFMAs
        if (active) {
            const float sg = sign(unit);
            auto at = [&](int offset) __attribute__((always_inline)) { return (LdsTr)(buf + offset); };
            bf16x8 d[3][2];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) d[q][kb] = split_tr_read(at(dp + q * 2 * DB + kb * 32), at(dp + q * 2 * DB + kb * 32 + 256));
            auto input = [&](int tap, int q, bf16x8 (&f)[2]) __attribute__((always_inline)) {
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const int off = q * 2 * XB + (tap / R * HW + tap % R) * 64 + cb * 32;
                    f[cb] = split_tr_read(at(xp[0] + off), at(xp[1] + off));
                }
            };
            bf16x8 f[3][2];
            input(0, 2, f[2]);
            input(0, 1, f[1]);
            input(0, 0, f[0]);
            static_for<0, S * R>([&](auto T) __attribute__((always_inline)) {
                constexpr int tap = decltype(T)::value;
                constexpr bool last = tap + 1 == S * R;
                floatx4 t[2][2];
                auto mul = [&](int qd, int qf, bool first) __attribute__((always_inline)) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb)
                            t[kb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[qd][kb], f[qf][cb], first ? floatx4{0.f, 0.f, 0.f, 0.f} : t[kb][cb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                };
                // the small products first: beside the leading pieces' only their sum is rounded
                if constexpr (SHORT) {                              // two of the products usually left out
                    mul(1, 2, true);
                    mul(2, 1, false);
                }
                mul(0, 2, !SHORT);
                if constexpr (!last) input(tap + 1, 2, f[2]);
                mul(1, 1, false);
                mul(0, 1, false);
                if constexpr (!last) input(tap + 1, 1, f[1]);
                mul(2, 0, false);
                mul(1, 0, false);
                // (SHORT: the two meet in an fp32 addition, as above)
                if constexpr (SHORT) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb)
                            t[kb][cb] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[0][kb], f[0][cb], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                } else {
                    mul(0, 0, false);
                }
                if constexpr (!last) input(tap + 1, 0, f[0]);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[tap][kb][cb][r] = __builtin_fmaf(t[kb][cb][r], sg, acc[tap][kb][cb][r]);
            });
        }
        if (unit + 1 - u0 == team.steps) break;
        if (TEAMS == 1 || unit + 1 < u1) Stage::stash(sd, sx, sign(unit + 1), lds + (unit + 1 - u0) % 2 * Stage::bytes(3));
        __syncthreads();                                     // (as often by a team of one tile less: not after the other's last)
    }
    if (TEAMS > 1)
        for (int i = u1 - u0; i + 1 < team.steps; ++i) __syncthreads();         // a team without tiles
    if (!team.join(acc, active, wave, lane, lds_all)) return;

    // D layout of a 16x16 block: column (c) = lane % 16, row (k) = 4*(lane/16) + r: four consecutive output channels, one 16-byte store,
    // the lanes' side by side
    const int k32 = kt * 64 + kh * 32, c32 = cg * 64 + ch * 32;
    float *pbase = part + (size_t)blockIdx.x * A.K * A.C * (S * R);
    auto element = [&](int k, int c, int tap) __attribute__((always_inline)) {
        return pbase + (((size_t)(k / kBlk) * CB + c / kBlk) * (S * R) + tap) * (kBlk * kBlk) + (c % kBlk) * kBlk + k % kBlk;
    };
    bool finite = true;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int k = k32 + kb * 16 + 4 * grp, c = c32 + cb * 16 + l16;
            if (k >= A.K || c >= A.C) continue;
#pragma unroll
            for (int tap = 0; tap < S * R; ++tap) {
                const floatx4 a = acc[tap][kb][cb];
                const float4 v = make_float4(a[0] * kSplitUnscale, a[1] * kSplitUnscale, a[2] * kSplitUnscale, a[3] * kSplitUnscale);
                finite = finite && split_finite(v);
                *reinterpret_cast<float4 *>(element(k, c, tap)) = v;
            }
        }
    // sums that values outside the range of the scaled pieces took part in
    if (__builtin_expect(__ballot(!finite) != 0, 0)) {
        split_lanes_fence();
        floatx16 redo[S * R];
        bww_redo<R, S, TH, TW, 1>(A, x, dy, k32, c32, team.first, team.last, redo);
        const int c = c32 + lane % 32;
        if (c >= A.C) return;
#pragma unroll
        for (int tap = 0; tap < S * R; ++tap)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k32 + 8 * (r / 4) + 4 * (lane / 32) + r % 4;
                if (k < A.K && !split_finite(*element(k, c, tap))) *element(k, c, tap) = redo[tap][r];
            }
    }
}

template <int R, int S, int TH, int TW, bool SHORT, bool BIG, int TEAMS>
__global__ __launch_bounds__(256 * TEAMS, 2) void bww_dense_wide_kernel(BwwArgs A, const float *__restrict__ x,
                                                                        const float *__restrict__ dy, float *__restrict__ part)
{
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    __shared__ __attribute__((aligned(16))) char lds[TEAMS * 2 * BwwWideStage<TH, TW>::bytes(3)];
    bww_dense_wide_body<R, S, TH, TW, SHORT, BIG, TEAMS>(A, x, dy, part, lds);
}

// Up to eight elements of a partial gradient once more, by the 64 lanes of a wavefront in 64 bits.  list: output channel - k32, input channel - c32 and tap,
// five, five and four bits, `count` of them
constexpr unsigned kBwwHalfFew = 8;
template <int TH, int TW>
__device__ __forceinline__ void bww_some(const BwwArgs &A, const float *x, const float *dy, int k32, int c32, const unsigned (&list)[kBwwHalfFew], unsigned count,
                                         int u0, int u1, double (&sum)[kBwwHalfFew])
{
    const int lane = threadIdx.x % kWave, p = lane % 32;
#pragma unroll
    for (unsigned i = 0; i < kBwwHalfFew; ++i) sum[i] = 0.;
#pragma unroll 2
    for (int unit = u0 + lane / 32; unit < u1; unit += 2) {
        const int tw = unit % A.tiles_w, th = unit / A.tiles_w % A.tiles_h, n = unit / A.tiles_w / A.tiles_h;
        const int oh = th * TH + p / TW, ow = tw * TW + p % TW;
#pragma unroll
        for (unsigned i = 0; i < kBwwHalfFew; ++i) {
            if (i >= count) break;
            const int k = k32 + (int)(list[i] & 31), c = c32 + (int)(list[i] >> 5 & 31), tap = (int)(list[i] >> 10);
            const int ih = oh - A.ph + tap / 3, iw = ow - A.pw + tap % 3;
            const bool in = p < TH * TW && oh < A.OH && ow < A.OW && ih >= 0 && ih < A.H && iw >= 0 && iw < A.W;
            const float d = dy[act_off(n, k / kBlk, in ? oh : 0, in ? ow : 0, A.K / kBlk, A.OH, A.OW) + k % kBlk];
            const float v = x[act_off(n, c / kBlk, in ? ih : 0, in ? iw : 0, A.C / kBlk, A.H, A.W) + c % kBlk];
            sum[i] += in ? (double)d * v : 0.;
        }
    }
#pragma unroll
    for (unsigned i = 0; i < kBwwHalfFew; ++i)
        for (int m = kWave / 2; m > 0; m /= 2) sum[i] += __shfl_xor(sum[i], m);
}

// The largest magnitude, in bits, of each of the 64 channels of x and of dy that a workgroup meets in tiles u0 .. u1-1: into most[0 ..], most[64 ..]
template <int TH, int TW>
__device__ __forceinline__ void bww_channels(const BwwArgs &A, const float *x, const float *dy, int kt, int cg, int u0, int u1, unsigned *most)
{
    using Stage = BwwWideStage<TH, TW>;
    if (threadIdx.x < 128) most[threadIdx.x] = 0;
    __syncthreads();
    unsigned mx[4] = {0u, 0u, 0u, 0u}, md[4] = {0u, 0u, 0u, 0u};
    typename Stage::Tile t;
    t.start(A, u0);
    auto meet = [](unsigned (&m)[4], float4 v) __attribute__((always_inline)) {
        m[0] = max(m[0], __float_as_uint(v.x) & 0x7fffffffu); m[1] = max(m[1], __float_as_uint(v.y) & 0x7fffffffu);
        m[2] = max(m[2], __float_as_uint(v.z) & 0x7fffffffu); m[3] = max(m[3], __float_as_uint(v.w) & 0x7fffffffu);
    };
#pragma unroll 4
    for (int unit = u0; unit < u1; ++unit) {
        float4 sd[2], sx[4];
        Stage::fetch_dy(A, dy, kt, t, sd);
        Stage::fetch_x(A, x, cg, t, sx);
        t.step(A);
        meet(md, sd[0]); meet(md, sd[1]);
        meet(mx, sx[0]); meet(mx, sx[1]); meet(mx, sx[2]); meet(mx, sx[3]);
    }
    const int q = threadIdx.x % 16 * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        atomicMax(most + q + i, mx[i]);
        atomicMax(most + 64 + q + i, md[i]);
    }
    __syncthreads();
}

// The same with two f16 pieces (st_split.hpp) where a workgroup has many tiles (kBwwHalfTiles): three products instead of six.  N = 32, half zeros, us:
// 256->256 @56 478 -> 353 (335 TFLOP/s), 512->512 @28 529 -> 375, 128->256 @56 246 -> 191, 64->64 @224 518 -> 425.  Bound: issue, half of it vector
// instructions (800 beside the 216 matrix instructions of a pair of tiles: splitting them, their addresses, joining the sums).  Workgroups take two tiles
// at a time, 64 pixels a sum, so that sums join half as often: what the pieces leave out (7.5e-8 of the norm) is less than what that saves.
// The registers are full (144 sums, 32 of a tap, 48 operands), so a pair is staged in three steps of 16 registers, each asked for three taps before
// it is split: the halo of its first tile into the third of three buffers that take turns, both dy tiles into the second pair of buffers, the halo
// of the second tile into the first buffer when this pair is done (two barriers a pair).  (24 registers, two steps: 20 spilled, 345 -> 372 us.)
// A tap of a tile is three groups of four instructions; the large and the small products have a sum each.
// False where the workgroup has to do all its tiles on bf16 pieces, instead or again.  All workgroups run at once, so the launch takes as long as the
// slowest: fp32 multiply-adds for a block with a single gradient that the pieces cannot give took 1300 us (below).  Instead: where fewer than four
// fifths of the sampled values of an operand are within 2^6 of the largest, so that values outside the pieces' range are to be expected, bf16
// pieces from the start; else a few gradients are computed one by one, those of channels without values are zeros (padding, ReLU: any lost value of the other
// operand makes them suspect), and only for more all tiles are done again.  us, bf16 pieces : fp32 multiply-adds : now, 16 x 256->256 @56 normal values
// 330 : 237 : 237, Laplace 304 : - : 250, 3 and 2 degrees of freedom 320 : - : 307, 294 : 1306 : 292, log-normal 2 294 : 1304 : 291, one in 10^4 100 times as
// large 289 : 1394 : 481, one in 10^4 2^-40 as large 291 : 203 : 241, all between 2^-40 and 1 305 : 1410 : 328; 13 of 16 channels zero,
// 32 x 128->64 @224 921 : 7446 : 899, 16->64 439 : 1598 : 430.
// Every thread makes the call.
template <int TH, int TW>
constexpr int kBwwHalfLds = 12 * BwwWideStage<TH, TW>::XB + 16 * BwwWideStage<TH, TW>::DB;
template <int TH, int TW>
__device__ __forceinline__ bool bww_dense_half_body(const BwwArgs &A, const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, char *lds)
{
    constexpr int R = 3, S = 3, TAPS = R * S;
    using Stage = BwwWideStage<TH, TW>;
    constexpr int HW = Stage::HW, TP = TH * TW, XB = Stage::XB, DB = Stage::DB, XBUF = 4 * XB, DBUF = 4 * DB;
    static_assert(kBwwHalfLds<TH, TW> == 3 * XBUF + 4 * DBUF, "three halos, four dy tiles");
    unsigned *misc = reinterpret_cast<unsigned *>(lds);         // before the first tile and after the last

    // the wavefront index is the same in every lane: kept in a scalar register, and with it every tile coordinate
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l16 = lane % 16, grp = lane / 16;
    const int kh = wave % 2, ch = wave / 2;
    const int split = blockIdx.x;
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;
    const int CB = A.C / kBlk, KB = A.K / kBlk;
    const bool active = kt * 64 + kh * 32 < A.K && cg * 64 + ch * 32 < A.C;

    const int u0 = (int)((long long)A.units * split / A.splits);
    const int u1 = (int)((long long)A.units * (split + 1) / A.splits);

    // a sample for the scales: the first pixels of 16 tiles
    int xe, de;
    {
        const int slot = threadIdx.x / 16, q = threadIdx.x % 16;
        const int u = u0 + (int)((long long)(u1 - u0) * slot / 16);
        const int tw = u % A.tiles_w, th = u / A.tiles_w % A.tiles_h, n = u / A.tiles_w / A.tiles_h;
        const int cb = min(cg * 4 + q / 4, CB - 1), kb = min(kt * 4 + q / 4, KB - 1);
        const float4 vx = *reinterpret_cast<const float4 *>(x + act_off(n, cb, min(th * TH, A.H - 1), min(tw * TW, A.W - 1), CB, A.H, A.W) + q % 4 * 4);
        const float4 vd = *reinterpret_cast<const float4 *>(dy + act_off(n, kb, th * TH, tw * TW, KB, A.OH, A.OW) + q % 4 * 4);
        const unsigned mx = wave_max(half_magnitude(vx)), md = wave_max(half_magnitude(vd));
        auto filled = [](float4 v) __attribute__((always_inline)) {             // values of the wavefront that are not zero
            return (unsigned)(__popcll(__ballot(v.x != 0.f)) + __popcll(__ballot(v.y != 0.f)) + __popcll(__ballot(v.z != 0.f)) + __popcll(__ballot(v.w != 0.f)));
        };
        auto over4 = [&](int at) __attribute__((always_inline)) { return misc[at] + misc[at + 1] + misc[at + 2] + misc[at + 3]; };
        const unsigned fx = filled(vx), fd = filled(vd);
        if (lane == 0) { misc[wave] = mx; misc[4 + wave] = md; misc[8 + wave] = fx; misc[12 + wave] = fd; }
        __syncthreads();
        const unsigned some_x = over4(8), some_d = over4(12);
        const unsigned bits_x = max(max(misc[0], misc[1]), max(misc[2], misc[3])), bits_d = max(max(misc[4], misc[5]), max(misc[6], misc[7]));
        xe = __builtin_amdgcn_readfirstlane(half_exponent(bits_x, kHalfTopInput));
        de = __builtin_amdgcn_readfirstlane(half_exponent(bits_d, kHalfTopInput));
        // those within 2^6 of the largest
        auto near = [](float4 v, unsigned bits) __attribute__((always_inline)) {
            const unsigned least = max(bits, (6u << 23) + 1) - (6u << 23);
            return (unsigned)(__popcll(__ballot(half_magnitude(v.x) >= least)) + __popcll(__ballot(half_magnitude(v.y) >= least)) +
                              __popcll(__ballot(half_magnitude(v.z) >= least)) + __popcll(__ballot(half_magnitude(v.w) >= least)));
        };
        const unsigned nx = near(vx, bits_x), nd = near(vd, bits_d);
        if (lane == 0) { misc[16 + wave] = nx; misc[20 + wave] = nd; }
        __syncthreads();
        const bool few = some_x * some_d < (1u << 20) / 14;     // of 1024 x 1024 (kBwwHalfTiles)
        const bool wide = over4(16) * 5 < some_x * 4 || over4(20) * 5 < some_d * 4;
        __syncthreads();                                        // (misc is overwritten from here on)
        if (__builtin_amdgcn_readfirstlane((int)(few || wide))) return false;
    }
    floatx4 acc[TAPS][2][2];                            // [tap][16 k][16 c]
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[t][kb][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
    // (every other pair with the opposite sign: BwwDenseStage)
    auto sign = [](int pair) __attribute__((always_inline)) { return pair % 2 ? -1.f : 1.f; };
    typename Stage::Tile ta, tb;                                // the two tiles to ask for next
    ta.start(A, u0);
    tb = ta;
    // a second tile that does not exist: rows that no image of these sizes has, all zeros
    auto second = [&](int unit) __attribute__((always_inline)) {
        tb = ta;
        tb.step(A);
        if (unit >= u1) { tb.n = 0; tb.th = kBwwNoTileRow / TH; }
    };
    auto first = [&](int unit) __attribute__((always_inline)) {
        ta = tb;
        ta.step(A);
        if (unit >= u1) { ta.n = 0; ta.th = kBwwNoTileRow / TH; }
    };
    float4 sx[4], sda[2], sdb[2];
    unsigned lows_x = 0, lows_d = 0;                            // of the four channels of x and of dy that this thread stages
    char *const xlds = lds, *const dlds = lds + 3 * XBUF;
    Stage::fetch_x(A, x, cg, ta, sx);                           // (a split has at least one tile)
    lows_x += Stage::template stash_half<XB>(sx, 1.f, xe, xlds);
    second(u0 + 1);
    Stage::fetch_dy(A, dy, kt, ta, sda);
    Stage::fetch_dy(A, dy, kt, tb, sdb);
    Stage::fetch_x(A, x, cg, tb, sx);
    lows_d += Stage::template stash_half<DB>(sda, 1.f, de, dlds);
    lows_d += Stage::template stash_half<DB>(sdb, 1.f, de, dlds + DBUF);
    lows_x += Stage::template stash_half<XB>(sx, 1.f, xe, xlds + XBUF);
    __syncthreads();

    // operands: lane l takes channel l % 16 of a block and pixels 8*(l/16) .. +7 of the tile, four per transposing read, for which
    // it supplies the address of 8 bytes of pixel (l % 16) / 4 of the four
    int dp, xp[2];
    {
        const int px = grp * 8 + l16 / 4, chan = l16 % 4 * 8;
        dp = kh * DB + px * 64 + chan;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int p = min(px + i * 4, TP - 1);              // (the padding's dy is zero)
            xp[i] = ch * XB + (p / TW * HW + p % TW) * 64 + chan;
        }
    }
    int slot = 0;                                               // buffer of the pair's first tile; the second one's is the next
    for (int unit = u0, pair = 0;; unit += 2, ++pair) {
        const bool more = unit + 2 < u1;
        char *const tile[2] = {xlds + slot * XBUF, xlds + (slot + 1) % 3 * XBUF}, *const spare = xlds + (slot + 2) % 3 * XBUF;
        char *const dtile = dlds + pair % 2 * (2 * DBUF), *const dspare = dlds + (1 - pair % 2) * (2 * DBUF);
        // (no branches around what follows, also not for a last pair's successor or for wavefronts without channels of their own, which multiply
        // zeros: with them 20 to 40 registers are spilled)
        first(unit + 2);
        second(unit + 3);
        Stage::fetch_x(A, x, cg, ta, sx);                       // in flight during the first taps
        __builtin_amdgcn_sched_barrier(0);
        const float sg = sign(pair), nsg = sign(pair + 1);
        auto at = [&](int t, int offset) __attribute__((always_inline)) { return (LdsTr)(tile[t] + offset); };
        auto dat = [&](int t, int offset) __attribute__((always_inline)) { return (LdsTr)(dtile + t * DBUF + offset); };
        auto read = [&](LdsTr p0, LdsTr p1) __attribute__((always_inline)) { return __builtin_bit_cast(f16x8, split_tr_read(p0, p1)); };
        auto input = [&](int t, int tap, int q, f16x8 (&f)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int off = q * 2 * XB + (tap / R * HW + tap % R) * 64 + cb * 32;
                f[cb] = read(at(t, xp[0] + off), at(t, xp[1] + off));
            }
        };
        f16x8 d[2][2][2], f[2][2];                              // [tile][piece][16 k], [piece][16 c]
        auto taps = [&](auto First, auto Last) __attribute__((always_inline)) {
            static_for<decltype(First)::value, decltype(Last)::value>([&](auto T) __attribute__((always_inline)) {
                constexpr int tap = decltype(T)::value;
                floatx4 large[2][2], small[2][2];
                static_for<0, 2>([&](auto Tile) __attribute__((always_inline)) {
                    constexpr int t = decltype(Tile)::value;
                    constexpr int nt = 1 - t, ntap = t == 0 ? tap : tap + 1;            // whose input replaces this one's
                    auto mul = [&](int qd, int qf, floatx4 (&to)[2][2], bool first) __attribute__((always_inline)) {
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int cb = 0; cb < 2; ++cb)
                                to[kb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(d[t][qd][kb], f[qf][cb], first ? floatx4{0.f, 0.f, 0.f, 0.f} : to[kb][cb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    mul(0, 0, large, t == 0);
                    mul(1, 0, small, t == 0);
                    if constexpr (ntap < TAPS) input(nt, ntap, 0, f[0]);
                    mul(0, 1, small, false);
                    if constexpr (ntap < TAPS) input(nt, ntap, 1, f[1]);
                });
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            acc[tap][kb][cb][r] = __builtin_fmaf(__builtin_fmaf(small[kb][cb][r], 1.f / kHalfLow, large[kb][cb][r]), sg, acc[tap][kb][cb][r]);
                // (here, not behind the loop's end where the compiler would take it with 256 registers in scratch memory)
                asm volatile("" : "+v"(acc[tap][0][0]), "+v"(acc[tap][0][1]), "+v"(acc[tap][1][0]), "+v"(acc[tap][1][1]));
                __builtin_amdgcn_sched_barrier(0);
            });
        };
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) d[t][q][kb] = read(dat(t, dp + q * 2 * DB + kb * 32), dat(t, dp + q * 2 * DB + kb * 32 + 256));
        input(0, 0, 0, f[0]);
        input(0, 0, 1, f[1]);
        taps(std::integral_constant<int, 0>{}, std::integral_constant<int, 3>{});
        lows_x += Stage::template stash_half<XB>(sx, 1.f, xe, spare);
        Stage::fetch_dy(A, dy, kt, ta, sda);
        Stage::fetch_dy(A, dy, kt, tb, sdb);
        __builtin_amdgcn_sched_barrier(0);
        taps(std::integral_constant<int, 3>{}, std::integral_constant<int, 6>{});
        lows_d += Stage::template stash_half<DB>(sda, nsg, de, dspare);
        lows_d += Stage::template stash_half<DB>(sdb, nsg, de, dspare + DBUF);
        Stage::fetch_x(A, x, cg, tb, sx);
        __builtin_amdgcn_sched_barrier(0);
        taps(std::integral_constant<int, 6>{}, std::integral_constant<int, TAPS>{});
        if (!more) break;
        __syncthreads();                                        // every wavefront is done with the pair
        lows_x += Stage::template stash_half<XB>(sx, 1.f, xe, tile[0]);
        __syncthreads();
        slot = (slot + 2) % 3;
    }

    // Fours with a value below the pieces' range, of each four channels of x, then of dy, in the third halo buffer, which no one reads now.
    // Others may still be writing it, also the halo of a tile that does not exist: not before a barrier
    misc = reinterpret_cast<unsigned *>(xlds + (slot + 2) % 3 * XBUF);
    {
        if (__ballot((lows_x | lows_d) != 0) != 0) {
            lows_x += __shfl_xor(lows_x, 16); lows_x += __shfl_xor(lows_x, 32);
            lows_d += __shfl_xor(lows_d, 16); lows_d += __shfl_xor(lows_d, 32);
        }
        __syncthreads();
        if (lane < 16) { misc[wave * 32 + l16] = lows_x; misc[wave * 32 + 16 + l16] = lows_d; }
        __syncthreads();
    }
    auto safe = [&](int kb, int cb) __attribute__((always_inline)) {
        const int at_x = ch * 8 + cb * 4 + l16 / 4, at_d = 16 + kh * 8 + kb * 4 + grp;
        const unsigned lost = misc[at_x] + misc[32 + at_x] + misc[64 + at_x] + misc[96 + at_x] + misc[at_d] + misc[32 + at_d] + misc[64 + at_d] + misc[96 + at_d];
        return kHalfSafe * fminf(4.f * (float)lost / (float)((u1 - u0) * TP), 1.f);
    };

    // D layout of a 16x16 block: column (c) = lane % 16, row (k) = 4*(lane/16) + r: four consecutive output channels, one 16-byte store,
    // the lanes' side by side
    const int k32 = kt * 64 + kh * 32, c32 = cg * 64 + ch * 32, exponent = -(xe + de);
    float *pbase = part + (size_t)split * A.K * A.C * TAPS;
    auto element = [&](int k, int c, int tap) __attribute__((always_inline)) {
        return pbase + (((size_t)(k / kBlk) * CB + c / kBlk) * TAPS + tap) * (kBlk * kBlk) + (c % kBlk) * kBlk + k % kBlk;
    };
    bool finite = true;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int k = k32 + kb * 16 + 4 * grp, c = c32 + cb * 16 + l16;
            const float least = safe(kb, cb);
            auto finish = [&](float v) __attribute__((always_inline)) { return fabsf(v) < least ? __builtin_nanf("") : ldexpf(v, exponent); };
            if (!active || k >= A.K || c >= A.C) continue;
#pragma unroll
            for (int tap = 0; tap < TAPS; ++tap) {
                const floatx4 a = acc[tap][kb][cb];
                const float4 v = make_float4(finish(a[0]), finish(a[1]), finish(a[2]), finish(a[3]));
                finite = finite && split_finite(v);
                *reinterpret_cast<float4 *>(element(k, c, tap)) = v;
            }
        }

    // Gradients that are infinite (values above the pieces' range took part in them) or so small that lost values may matter: a few are
    // computed one by one; if there are more, those of channels without any values are zeros; and for more than a few others the workgroup
    // starts again on bf16 pieces
    unsigned *const votes = misc + 128, *const most = misc + 256;
    auto vote = [&](unsigned n) __attribute__((always_inline)) {
        if (lane == 0) votes[wave] = n;
        __syncthreads();
        const unsigned m = max(max(votes[0], votes[1]), max(votes[2], votes[3]));
        __syncthreads();                                        // (the words, and all others here, are written again)
        return (unsigned)__builtin_amdgcn_readfirstlane((int)m);
    };
    // what(whether it is one of these, ...) of the lane's outputs, one of each lane at a time; those of three taps are asked for together
    auto each = [&](auto what) __attribute__((always_inline)) {
#pragma unroll 1
        for (int t = 0; t < TAPS / 3 * 4; ++t) {
            const int kl = t / 2 % 2 * 16 + 4 * grp, cl = t % 2 * 16 + l16;
            const bool exists = k32 + kl < A.K && c32 + cl < A.C;
            float *at[3];
            float4 v[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                at[i] = element(exists ? k32 + kl : k32, exists ? c32 + cl : c32, t / 4 * 3 + i);
                v[i] = *reinterpret_cast<const float4 *>(at[i]);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                what(exists && !split_finite(v[i].x), kl, cl, t / 4 * 3 + i, at[i]);
                what(exists && !split_finite(v[i].y), kl + 1, cl, t / 4 * 3 + i, at[i] + 1);
                what(exists && !split_finite(v[i].z), kl + 2, cl, t / 4 * 3 + i, at[i] + 2);
                what(exists && !split_finite(v[i].w), kl + 3, cl, t / 4 * 3 + i, at[i] + 3);
            }
        }
    };
    auto count = [&]() __attribute__((always_inline)) {
        unsigned n = 0;
        each([&](bool again, int, int, int, float *) __attribute__((always_inline)) { n += (unsigned)__popcll(__ballot(again)); });
        return n;
    };
    unsigned open = 0;
    if (__builtin_expect(__ballot(!finite) != 0, 0)) open = count();
    unsigned worst = vote(open);
    if (__builtin_expect(worst == 0, 1)) return true;
    if (worst > kBwwHalfFew) {
        bww_channels<TH, TW>(A, x, dy, kt, cg, u0, u1, most);
        unsigned above = max(most[lane], most[64 + lane]);
        const bool all_finite = __ballot(above >= 0x7f800000u) == 0;            // (0 * inf is not 0)
        if (open != 0 && all_finite)
            each([&](bool again, int kl, int cl, int, float *at) __attribute__((always_inline)) {
                if (again && (most[ch * 32 + cl] == 0 || most[64 + kh * 32 + kl] == 0)) *at = 0.f;
            });
        if (open != 0) open = count();
        worst = vote(open);
    }
    if (worst > kBwwHalfFew) return false;
    if (open != 0) {
        unsigned list[kBwwHalfFew] = {}, n = 0;
        each([&](bool again, int kl, int cl, int tap, float *) __attribute__((always_inline)) {
            for (unsigned long long m = __ballot(again); m != 0; m &= m - 1, ++n) {
                const int l = __builtin_ctzll(m);
                const unsigned entry = (unsigned)(__builtin_amdgcn_readlane(kl, l) | __builtin_amdgcn_readlane(cl, l) << 5 | tap << 10);
#pragma unroll
                for (unsigned i = 0; i < kBwwHalfFew; ++i) list[i] = n == i ? entry : list[i];
            }
        });
        double sum[kBwwHalfFew];
        bww_some<TH, TW>(A, x, dy, k32, c32, list, open, u0, u1, sum);
        split_lanes_fence();                                    // (other lanes wrote what the first one replaces)
#pragma unroll
        for (unsigned i = 0; i < kBwwHalfFew; ++i)
            if (i < open && lane == 0) *element(k32 + (int)(list[i] & 31), c32 + (int)(list[i] >> 5 & 31), (int)(list[i] >> 10)) = (float)sum[i];
    }
    return true;
}

template <int TH, int TW>
__global__ __launch_bounds__(256, 2) void bww_dense_half_kernel(BwwArgs A, const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part)
{
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    constexpr int LDS = kBwwHalfLds<TH, TW>;
    static_assert(LDS >= 2 * BwwWideStage<TH, TW>::bytes(3) && 2 * LDS <= 160 * 1024, "either form in one array, two workgroups a compute unit");
    __shared__ __attribute__((aligned(16))) char lds[LDS];
    if (!bww_dense_half_body<TH, TW>(A, x, dy, part, lds)) bww_dense_wide_body<3, 3, TH, TW, false, false, 1>(A, x, dy, part, lds);
}

// ------------------------------------------------------------------------------------------
// 1x1 layers (unit stride, no padding): dw[k][c] = sum over all N*H*W pixels of dy[p][k] * x[p][c],
// a matrix product with the pixels as the reduction dimension (Sec. 5.2 of the paper).  Pixels are
// numbered across the minibatch and cut into chunks of PWP; `units` counts chunks.
// ------------------------------------------------------------------------------------------
constexpr int kPwP = 32;            // pixels per staged chunk

// KJ x CI blocks of 32 x 32 elements of a 1x1 partial gradient once more with fp32 multiply-adds on the matrix cores (as
// bww_redo): `count` pixels of the minibatch from pixel (n, p) on
template <int KJ, int CI>
__device__ __forceinline__ void pw_bww_redo(const BwwArgs &A, const float *x, const float *dy, int k0, int c0, int n, int p, long long count,
                                            floatx16 (&acc)[KJ][CI])
{
    const int lane = threadIdx.x % kWave, l32 = lane % 32, half = lane / 32;
    const int HW = A.H * A.W;
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
        for (int i = 0; i < CI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
    p += half;
#pragma unroll 4
    for (long long q = 0; q < count; q += 2) {
        while (p >= HW) { p -= HW; ++n; }
        const bool in = q + half < count && n < A.N;
        float d[KJ], xv[CI];
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const int k = min(k0 + j * 32 + l32, A.K - 1);                      // (past the end: not stored)
            d[j] = dy[in ? (((size_t)n * (A.K / kBlk) + k / kBlk) * HW + p) * kBlk + k % kBlk : 0];
        }
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            const int c = min(c0 + i * 32 + l32, A.C - 1);
            xv[i] = x[in ? (((size_t)n * (A.C / kBlk) + c / kBlk) * HW + p) * kBlk + c % kBlk : 0];
        }
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < CI; ++i)
                acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? d[j] : 0.f, in ? xv[i] : 0.f, acc[j][i], 0, 0, 0);
        p += 2;
    }
}

// Dense, on bf16 pieces (st_split.hpp): workgroup = CW input channels x KW output channels (128 or 64 each).  Its eight
// wavefronts are two teams of four that take alternate chunks of P pixels and add up their sums through LDS at the end: half
// the partial gradients of as many separate workgroups (on 512->2048 @7 they are 33 MB written and read again, as
// long as the arithmetic).  The four wavefronts of a team are a 2 x 2 grid of (KW/2) x (CW/2) sub-tiles of 32x32 MFMA blocks
// (rows = output channels, columns = input channels, reduction = 16 pixels); the team's next chunk is fetched into
// registers while the current one is multiplied.  128 x 128 uses a staged pixel for four blocks; layers with only 64
// channels on a side get the narrower tile (no padded blocks) and chunks of 64 pixels, so that there are as many
// matrix instructions between two barriers.  Between two barriers one team multiplies while the other splits and stashes
// its next chunk, so the matrix cores and the vector ALUs work at the same time.  The products of the leading pieces go straight
// to the sums; the others have accumulators of their own, which join the sums once per chunk, and the sums change sign
// there.  (6x56x56 pixels, 4 % non-zero products, 16 and 64 channels, error: 1.2e-7 of the norm with one accumulator for all
// products and the partial sums added up in 32 bits, 6e-8 to 7e-8 now.)
template <int CW, int KW, int P>
__global__ __launch_bounds__(512, 2) void pw_bww_dense_kernel(BwwArgs A, const float *__restrict__ x,
                                                              const float *__restrict__ dy, float *__restrict__ part)
{
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    constexpr int CI = CW / 64, KJ = KW / 64;           // 32-channel blocks of a wavefront
    constexpr int NX = P * (CW / 4) / 256, ND = P * (KW / 4) / 256;
    constexpr int XB = CW * P * 2, DB = KW * P * 2;     // bytes of one piece of a chunk: [32-channel block][pixel][32 channels]
    constexpr int TEAM = 3 * (XB + DB), SUMS = 256 * CI * KJ * 64;
    static_assert(SUMS <= 2 * TEAM, "the second team's sums go through the same LDS");
    extern __shared__ __attribute__((aligned(16))) char pw_lds[];       // 2 * TEAM bytes

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l32 = lane % 32, half = lane / 32;
    const int team = wave / 4, wk = wave % 2, wc = wave / 2 % 2;
    const int split = blockIdx.x;
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;
    const int CB = A.C / kBlk, KB = A.K / kBlk;
    const int HW = A.H * A.W;
    char *const xs = pw_lds + team * TEAM, *const ds = xs + 3 * XB;
    const bool active = kt * KW + wk * (KW / 2) < A.K && cg * CW + wc * (CW / 2) < A.C;

    floatx16 sum[KJ][CI];
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
        for (int i = 0; i < CI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[j][i][r] = 0.f;

    const int u0 = (int)((long long)A.units * split / A.splits);
    const int u1 = (int)((long long)A.units * (split + 1) / A.splits);

    // staging slots of this thread: slot = (pixel, 4 channels).  (image, pixel) of a chunk's first pixel is
    // carried from chunk to chunk (one 64-bit division per workgroup instead of one per slot and chunk); a
    // slot's pixel is that plus its offset, wrapped into the following images.
    float4 rx[NX], rd[ND];
    const int t256 = threadIdx.x % 256;
    int n0 = (int)((long long)(u0 + team) * P / HW), p0 = (int)((long long)(u0 + team) * P % HW);
    auto fetch = [&]() __attribute__((always_inline)) {      // the chunk that starts at (n0, p0); zeros past the last image
#pragma unroll
        for (int jj = 0; jj < NX + ND; ++jj) {
            const bool isx = jj < NX;
            const int idx = (isx ? jj : jj - NX) * 256 + t256, quads = (isx ? CW : KW) / 4;
            const int pix = idx / quads, q = idx % quads;
            const int blk = isx ? cg * (CW / kBlk) + (q >> 2) : kt * (KW / kBlk) + (q >> 2);
            int n = n0, p = p0 + pix;
            while (p >= HW) { p -= HW; ++n; }
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (n < A.N && blk < (isx ? CB : KB))
                v = *reinterpret_cast<const float4 *>((isx ? x : dy) + (((size_t)n * (isx ? CB : KB) + blk) * HW + p) * kBlk + (q & 3) * 4);
            if (isx) rx[isx ? jj : 0] = v;
            else rd[isx ? 0 : jj - NX] = v;
        }
        p0 += 2 * P;
        while (p0 >= HW) { p0 -= HW; ++n0; }
    };
    auto stash = [&](bool flip) __attribute__((always_inline)) {
#pragma unroll
        for (int jj = 0; jj < NX + ND; ++jj) {
            const bool isx = jj < NX;
            const int idx = (isx ? jj : jj - NX) * 256 + t256, quads = (isx ? CW : KW) / 4;
            const int pix = idx / quads, q = idx % quads;
            bf16x4 w[3];
            split4(isx ? rx[isx ? jj : 0] : rd[isx ? 0 : jj - NX], !isx && flip ? -kSplitScale : kSplitScale, w);
            char *dst = (isx ? xs : ds) + (q >> 3) * (P * 64) + pix * 64 + (q & 7) * 8;
#pragma unroll
            for (int i = 0; i < 3; ++i) *reinterpret_cast<bf16x4 *>(dst + i * (isx ? XB : DB)) = w[i];
        }
    };

    // this lane's address for the first four pixels of its half of step 0
    const int lane_off = (half * 8 + lane % 16 / 4) * 64 + split_tr_lane(lane);
    const LdsTr xp = (LdsTr)(xs + wc * CI * (P * 64) + lane_off), dp = (LdsTr)(ds + wk * KJ * (P * 64) + lane_off);

    // Phases of team 0: multiply chunk 0, stash 1, multiply 1, ...; of team 1, one behind: stash 0, multiply 0, ...
    const int rounds = (u1 - u0 + 1) / 2;               // the same for both teams (barriers); the last may be one team's only
    auto flip = [&](int it) __attribute__((always_inline)) { return (it + split + team) % 2 != 0; };
    const bool apart = rounds * P <= kSplitApartPixels;
    if (u0 + team < u1) fetch();
    if (team == 0) stash(flip(0));                      // (a workgroup has at least one chunk)
    __syncthreads();
    auto multiply = [&](auto A) __attribute__((always_inline)) {
        constexpr bool APART = decltype(A)::value;
        floatx16 block[KJ][CI];
#pragma unroll
        for (int s = 0; s < P / 16; ++s) {
            bf16x8 d[KJ][3], f[CI][3];
#pragma unroll
            for (int j = 0; j < KJ; ++j)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int off = (j * (P * 64) + q * DB + s * 1024) / 8;
                    d[j][q] = split_tr_read(dp + off, dp + off + 32);
                }
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int off = (i * (P * 64) + q * XB + s * 1024) / 8;
                    f[i][q] = split_tr_read(xp + off, xp + off + 32);
                }
            if (s > 0 && s % 2 == 0 && !APART) {            // a block is 32 pixels
#pragma unroll
                for (int j = 0; j < KJ; ++j)
#pragma unroll
                    for (int i = 0; i < CI; ++i) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum[j][i][r] += block[j][i][r];
                    }
            }
            constexpr int ta[5] = {2, 0, 1, 1, 0}, tb[5] = {0, 2, 1, 0, 1};            // smallest products first
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int j = 0; j < KJ; ++j)
#pragma unroll
                    for (int i = 0; i < CI; ++i)
                        block[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[j][ta[t]], f[i][tb[t]],
                                                                              (APART ? s == 0 : s % 2 == 0) && t == 0 ? floatx16{} : block[j][i], 0, 0, 0);
            // (left to itself the compiler moves these up and the next step's reads down: 256->64 @56 36.6 -> 37.5)
            if constexpr (KJ * CI > 1) __builtin_amdgcn_sched_barrier(0);
            auto leading = [&](floatx16 (&to)[KJ][CI]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < KJ; ++j)
#pragma unroll
                    for (int i = 0; i < CI; ++i) to[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[j][0], f[i][0], to[j][i], 0, 0, 0);
            };
            if constexpr (APART) leading(sum);
            else leading(block);
        }
        // the block joins the sum, which changes sign (with the dy of the team's next chunk)
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[j][i][r] = -sum[j][i][r] - block[j][i][r];
    };
    for (int ph = 0; ph < 2 * rounds; ++ph) {
        const int it = (ph + (team == 0 ? ph % 2 : 0)) / 2, unit = u0 + 2 * it + team;
        if (ph % 2 != team) {
            if (unit < u1) stash(flip(it));
        } else if (unit < u1) {
            if (unit + 2 < u1) fetch();                 // in flight during the MFMAs below
            if (active) {
                if (apart) multiply(std::true_type{});              // uniform
                else multiply(std::false_type{});
            }
        }
        __syncthreads();
    }

    // the second team's sums join the first's: [register][thread of the team]
    const float scale = flip((u1 - u0 - team + 1) / 2) ? -kSplitUnscale : kSplitUnscale;       // (after that many chunks)
    float *red = reinterpret_cast<float *>(pw_lds) + t256;
    if (team == 1) {
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[((j * CI + i) * 16 + r) * 256] = sum[j][i][r] * scale;
    }
    __syncthreads();
    if (team == 1 || !active) return;

    // D[row = k][column = c]: column = lane % 32, row = 8*(r/4) + 4*(lane/32) + r%4
    float *pbase = part + (size_t)split * A.K * A.C;
    auto element = [&](int k, int c) __attribute__((always_inline)) {
        return pbase + ((size_t)(k / kBlk) * CB + c / kBlk) * (kBlk * kBlk) + (c % kBlk) * kBlk + k % kBlk;
    };
    bool finite = true;
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            const int c = cg * CW + wc * (CW / 2) + i * 32 + l32;
            if (c >= A.C) continue;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const int k = kt * KW + wk * (KW / 2) + j * 32 + 8 * gq + 4 * half;
                if (k >= A.K) continue;
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = fmaf(sum[j][i][4 * gq + r], scale, red[((j * CI + i) * 16 + 4 * gq + r) * 256]);
                    finite = finite && split_finite(v[r]);
                }
                *reinterpret_cast<float4 *>(element(k, c)) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    // sums that values outside the range of the scaled pieces took part in
    if (__builtin_expect(__ballot(!finite) != 0, 0)) {
        const int k0 = kt * KW + wk * (KW / 2), c0 = cg * CW + wc * (CW / 2);
        const long long first = (long long)u0 * P, end = (long long)A.N * HW, last = (long long)u1 * P;
        pw_bww_redo<KJ, CI>(A, x, dy, k0, c0, (int)(first / HW), (int)(first % HW), (last < end ? last : end) - first, sum);
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < CI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int k = k0 + j * 32 + 8 * (r / 4) + 4 * half + r % 4, c = c0 + i * 32 + l32;
                    if (k < A.K && c < A.C && !split_finite(*element(k, c))) *element(k, c) = sum[j][i][r];
                }
    }
}

// Zero-skipping: lane = KPL output channels (k, k+64, ...), wavefront = 8 input channels, workgroup =
// 8 wavefronts = 64 input channels, as in bww_sparse_kernel but with KPL accumulators per tested
// element instead of R*S: without taps, the number of multiply-adds a zero saves is the number of
// output channels a lane owns (T = K/64 up to 4), the 1x1 analogue of T = Q/V in Sec. 5.2.
template <int KPL>
__global__ __launch_bounds__(512, 4) void pw_bww_sparse_kernel(BwwArgs A, const float *__restrict__ x,
                                                               const float *__restrict__ dy,
                                                               float *__restrict__ part)
{
    constexpr int P = kPwP, CH = 8, GP = 4, KW = 64 * KPL;
    if (deselected(A.sel, A.want)) return;              // uniform over the grid, before any barrier
    __shared__ __attribute__((aligned(16))) float dyT[P * KW];
    __shared__ __attribute__((aligned(16))) float xT[P * 64];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int split = blockIdx.x;
    const int kt = blockIdx.y / A.cgroups, cg = blockIdx.y % A.cgroups;     // kt: groups of KW, cg: of 64
    const int CB = A.C / kBlk, KB = A.K / kBlk;
    const int cbl = wave >> 1, h = wave & 1;
    const int cb = cg * 4 + cbl;
    const bool wave_active = cb < CB;
    const int HW = A.H * A.W;

    float acc[CH][KPL];
#pragma unroll
    for (int ci = 0; ci < CH; ++ci)
#pragma unroll
        for (int j = 0; j < KPL; ++j) acc[ci][j] = 0.f;

    const int u0 = (int)((long long)A.units * split / A.splits);
    const int u1 = (int)((long long)A.units * (split + 1) / A.splits);
    const int mpix = lane >> 4, mch = lane & 15;

    // (image, pixel) of the chunk's first pixel, carried from chunk to chunk: one 64-bit division per
    // workgroup instead of one per staged float4
    int n0 = (int)((long long)u0 * P / HW), p0 = (int)((long long)u0 * P % HW);
    auto locate = [&](int pix, int &n, int &p) __attribute__((always_inline)) {
        n = n0;
        p = p0 + pix;
        while (p >= HW) { p -= HW; ++n; }
        return n < A.N;
    };
    // A thread's 16-byte pieces of a chunk (KPL of dy, one of x; zeros past the last image and beyond the channel
    // count) are asked for while the previous chunk is worked on and written to LDS after it: with load, wait
    // and write in turn a chunk of 32 pixels cost KPL + 1 memory round trips, more than its arithmetic.
    constexpr int NDY = P * (KW / 4) / 512;
    static_assert(NDY * 512 == P * (KW / 4) && P * 16 == 512, "one x piece and KPL dy pieces per thread");
    float4 sdy[NDY], sxv;
    auto fetch = [&]() __attribute__((always_inline)) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                   // (slot arithmetic redone per chunk, not kept in registers)
#pragma unroll
        for (int i = 0; i < NDY; ++i) {
            const int idx = tid + i * 512;
            const int pix = idx / (KW / 4), q = idx % (KW / 4);
            const int kb = kt * (KW / kBlk) + (q >> 2);
            int n, p;
            sdy[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (locate(pix, n, p) && kb < KB)
                sdy[i] = *reinterpret_cast<const float4 *>(dy + (((size_t)n * KB + kb) * HW + p) * kBlk + (q & 3) * 4);
        }
        {
            const int pix = tid >> 4, q = tid & 15;
            const int cbq = cg * 4 + (q >> 2);
            int n, p;
            sxv = make_float4(0.f, 0.f, 0.f, 0.f);
            if (locate(pix, n, p) && cbq < CB)
                sxv = *reinterpret_cast<const float4 *>(x + (((size_t)n * CB + cbq) * HW + p) * kBlk + (q & 3) * 4);
        }
        p0 += P;
        while (p0 >= HW) { p0 -= HW; ++n0; }
    };
    if (u0 < u1) fetch();
    for (int unit = u0; unit < u1; ++unit) {
        __syncthreads();                                // every wavefront is done with the previous chunk
        {
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int i = 0; i < NDY; ++i) *reinterpret_cast<float4 *>(dyT + (tid + i * 512) * 4) = sdy[i];   // = [pix][q*4]
            *reinterpret_cast<float4 *>(xT + tid * 4) = sxv;
        }
        __syncthreads();
        if (unit + 1 < u1) fetch();                     // in flight during this chunk's work
        if (!wave_active) continue;

        // accumulators of channels 2i + 1 and 2i in (even, odd) register pairs, as in bww_sparse_kernel: never
        // the parity of the channel's tested value
        typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int ci = 0; ci < CH; ci += 2)
#pragma unroll
            for (int q = 0; q < KPL; ++q) {
                f2 pr = {acc[ci + 1][q], acc[ci][q]};
                asm volatile("" : "+v"(pr));
                acc[ci + 1][q] = pr.x;
                acc[ci][q] = pr.y;
            }

        float mnext = xT[mpix * 64 + cbl * 16 + mch];        // mask values are read one group ahead
        for (int g0 = 0; g0 < P; g0 += GP) {
            const float mval = mnext;
            if (g0 + GP < P) mnext = xT[(g0 + GP + mpix) * 64 + cbl * 16 + mch];
            const unsigned long long m64 = __builtin_amdgcn_ballot_w64(mval != 0.f);
            const unsigned mlo = (unsigned)m64, mhi = (unsigned)(m64 >> 32);
            if ((mlo | mhi) == 0u) continue;
            float dyw[GP][KPL];
#pragma unroll
            for (int j = 0; j < GP; ++j)
#pragma unroll
                for (int q = 0; q < KPL; ++q) dyw[j][q] = dyT[(g0 + j) * KW + q * 64 + lane];
            const float4 *xq = reinterpret_cast<const float4 *>(xT + g0 * 64 + cbl * 16 + h * CH);
            float4 xlo = xq[0], xhi = xq[1];
            __builtin_amdgcn_s_waitcnt(0xC07F);
            static_for<0, GP>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = decltype(J)::value;
                float4 nlo = xlo, nhi = xhi;
                if constexpr (j + 1 < GP) {
                    nlo = xq[(j + 1) * 16];
                    nhi = xq[(j + 1) * 16 + 1];
                }
                const float xv[CH] = {xlo.x, xlo.y, xlo.z, xlo.w, xhi.x, xhi.y, xhi.z, xhi.w};
                const unsigned mw = (j < 2) ? mlo : mhi;
                constexpr int sh = (j % 2) * 16;
                const unsigned bits = (mw >> sh) >> (h * CH) & 0xFFu;
                if (__builtin_expect(bits != 0u, 1)) {
                    static_for<0, CH>([&](auto CI) __attribute__((always_inline)) {
                        constexpr int ci = decltype(CI)::value;
                        if (__builtin_expect((bits & (1u << ci)) != 0u, 1)) {
#pragma unroll
                            for (int q = 0; q < KPL; ++q) acc[ci][q] = fmaf(xv[ci], dyw[j][q], acc[ci][q]);
                        }
                    });
                }
                if constexpr (j + 1 < GP) __builtin_amdgcn_s_waitcnt(0xC07F);
                xlo = nlo;
                xhi = nhi;
            });
        }
    }

    if (wave_active) {
        float *pbase = part + (size_t)split * A.K * A.C;
#pragma unroll
        for (int q = 0; q < KPL; ++q) {
            const int k = kt * KW + q * 64 + lane;
            if (k >= A.K) continue;
            if (!A.swapped) {
                float *p = pbase + ((size_t)(k / kBlk) * CB + cb) * (kBlk * kBlk) + (h * CH) * kBlk + k % kBlk;
#pragma unroll
                for (int ci = 0; ci < CH; ++ci) p[ci * kBlk] = acc[ci][q];
            } else {            // exchanged operands: block [cb][k block] of the layer, element [k % 16][h*8 + ci]
                float4 *p = reinterpret_cast<float4 *>(pbase + ((size_t)cb * KB + k / kBlk) * (kBlk * kBlk) +
                                                       (k % kBlk) * kBlk + h * CH);
                p[0] = make_float4(acc[0][q], acc[1][q], acc[2][q], acc[3][q]);
                p[1] = make_float4(acc[4][q], acc[5][q], acc[6][q], acc[7][q]);
            }
        }
    }
}

// dw[i] = sum over splits of part[s][i].  A workgroup owns 64 float4 outputs; its 16 wavefronts each
// add the splits s = w, w+16, ... (in that order) and wavefront 0 adds the 16 sums in wavefront
// order: a fixed tree, so the result does not depend on timing.  Layers with few filter elements
// and many splits (1x1, 64 x 64) would otherwise leave the sum to a handful of threads.
// dw may be the first partial itself (every element is read by the thread that later writes it).
// The grid is capped and workgroups stride over the outputs: a launch whose form was not selected
// (st_conv_bww_auto) then costs a few hundred workgroup dispatches instead of up to ten thousand.
// sp.f[form] = number of partial sums the form (0 tests x, 1 tests dy, 2 dense) leaves behind; with
// want = kAnyForm the launch adds up those of whichever form the sampled counts selected, else it
// belongs to the form `want` and does nothing when another one was selected.
// JOINED: those of the dense form are sums of two teams each (bww_teams) and are added up in 64 bits (an instance of its own: the loop beside the other
// costs every launch 0.2 to 0.4 us).
struct Splits3 { int f[3]; };
constexpr int kAnyForm = -2;
// part[first] + part[first + step] + ... below `splits` (n4 float4 apart), eight loads in flight at a time: each eight in
// pairs, their sums in 64 bits.  Added up one after the other in 32 bits, hundreds of partial sums round more often than
// the products in them (3x3 64->64, 4 x 30 x 28 pixels, 105 partial sums, 4 % non-zero products: error 9.9e-8 of the norm one
// after the other, 5.7e-8 here; v_mfma_f32_32x32x2_f32 and its 34 partial sums 9.6e-8).
struct Sum4 { double x, y, z, w; };
__device__ __forceinline__ Sum4 add_partials(const float4 *part, size_t n4, int first, int splits, int step)
{
    constexpr int BATCH = 8;
    Sum4 s = {0., 0., 0., 0.};
    int p = first;
    for (; p + (BATCH - 1) * step < splits; p += BATCH * step) {
        float4 v[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) v[b] = part[(size_t)(p + b * step) * n4];
        const float4 t = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    for (; p < splits; p += step) {
        const float4 v = part[(size_t)p * n4];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    return s;
}

// The same all in 64 bits, for sums of two teams each (bww_teams)
__device__ __forceinline__ Sum4 add_joined(const float4 *part, size_t n4, int first, int splits, int step)
{
    constexpr int BATCH = 8;
    Sum4 s = {0., 0., 0., 0.};
    for (int p = first; p < splits; p += BATCH * step) {
        float4 v[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) v[b] = part[(size_t)min(p + b * step, splits - 1) * n4];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            if (p + b * step >= splits) break;
            s.x += v[b].x; s.y += v[b].y; s.z += v[b].z; s.w += v[b].w;
        }
    }
    return s;
}

template <bool JOINED>
__global__ __launch_bounds__(1024) void bww_reduce_kernel(const float4 *part, float4 *dw, size_t n4, Splits3 sp,
                                                          const unsigned *sel, int want)
{
    int form = want < 0 ? 0 : want;
    if (sel) {
        form = selected_form(sel);
        if (want != kAnyForm && form != want) return;
    }
    const int splits = form == 0 ? sp.f[0] : form == 1 ? sp.f[1] : sp.f[2];
    auto add = [&](const float4 *p, int first, int step) __attribute__((always_inline)) {
        if constexpr (JOINED)
            if (form == 2) return add_joined(p, n4, first, splits, step);
        return add_partials(p, n4, first, splits, step);
    };
    // Few splits: a thread per output.  With few outputs as well, that many threads would wait for one load after the other;
    // there the 16 wavefronts of a workgroup share the partial sums (48->48 @12 stride 2, N = 4, 9 partial sums of 5184 float4:
    // 18.1 -> 16.4 us for the whole call; two partial sums of 576 are faster added up by one thread each, 17.5 : 18.4).
    if (splits <= 2 || (splits <= 16 && n4 >= 16384)) {
        for (size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 1024) {
            const Sum4 s = add(part + i, 0, 1);
            dw[i] = make_float4((float)s.x, (float)s.y, (float)s.z, (float)s.w);
        }
        return;
    }
    __shared__ Sum4 red[16][64];
    const int o = threadIdx.x % 64, sl = threadIdx.x / 64;
    const size_t nblk = (n4 + 63) / 64;
    for (size_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {       // uniform trip count per workgroup
        const size_t i = blk * 64 + o;
        Sum4 s = {0., 0., 0., 0.};
        if (i < n4)
            s = add(part + i, sl, 16);
        red[sl][o] = s;
        __syncthreads();
        if (sl == 0 && i < n4) {
            for (int q = 1; q < 16; ++q) {                  // (slices past the last partial sum are zero)
                const Sum4 v = red[q][o];
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
            dw[i] = make_float4((float)s.x, (float)s.y, (float)s.z, (float)s.w);
        }
        __syncthreads();                                    // red is rewritten by the next round
    }
}

constexpr size_t kReduceGrid = 512;          // workgroups of 1024 threads: two per compute unit
constexpr int kSparseTH = 7, kSparseTW = 8;     // unit stride: 224 ... 7 are multiples of 7; two double-buffered workgroups fit the LDS
constexpr int kSparseS2TH = 8, kSparseS2TW = 8; // stride 2, x tested
constexpr size_t kSparseLds = bww_async_lds_bytes<3, 3, kSparseTH, kSparseTW>();

// The zero-skipping unit-stride kernels use more dynamic LDS than a kernel may without being allowed to: once per
// device, outside any launch sequence a caller may be capturing into a graph later.
template <auto Kern>
hipError_t allow_dynamic_lds(size_t bytes)
{
    constexpr int kMaxDev = 64;
    static std::atomic<bool> allowed[kMaxDev] = {};         // (calls from several threads: at worst the attribute is set twice)
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    if (!allowed[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        allowed[dev] = true;
    }
    return hipSuccess;
}
BwwArgs make_args(const st_conv_desc &d, int TH, int TW, bool tiles_over_input);
BwwArgs sparse_args(const st_conv_desc &d);
BwwArgs dense_args(const st_conv_desc &d);
bool dense_wide(const st_conv_desc &d);
bool bww_s2(const st_conv_desc &d);
// dense unit-stride 3x3 kernel: 4 x 8 pixels, or 2 x 14 (two steps of 16 as well, 4 pixels of padding)
constexpr int kDenseTH = 4, kDenseTW = 8, kDenseWideTH = 2, kDenseWideTW = 14;
// stride-2 layers: 4x8 tiles keep the strided halo of the other operand (9x17 pixels x 64 channels) in LDS; the
// dense kernel takes 2x8 (5x17), whose next tile fits in registers beside its sums
constexpr int kS2TH = 4, kS2TW = 8, kDenseS2TH = 2, kDenseS2TW = 8;

constexpr int kBwwTargetWorkgroups = 512;
// dense launches of at most this many tiles, one or two for a workgroup, take the SHORT form (with a workgroup's time in its
// tiles it would cost 10 %: 512->512 @14, N = 4, 48 -> 53)
constexpr int kBwwShortUnits = 16;
// Unit-stride dense launches with this many tiles for a workgroup multiply f16 pieces.  In units of (1e-8 of the norm) squared T tiles err 54 + 2.9 T with
// bf16 pieces, whose sums join once a tile, and 130 + 1.3 T with f16 ones (256->256 @56, N = 32, half zeros, T = 98, 1.85e-7 : 1.61e-7, at 50 / 90 %
// 1.69e-7 : 1.62e-7, 128->256 @56, T = 49, 1.37e-7 : 1.36e-7, 512->512 @14, T = 28, 1.17e-7 : 1.28e-7).  Where few products are not zero
// sums have few terms to round, and a workgroup that samples that stays on bf16 pieces.  The line is at one in 14 (bf16 : f16, 1e-8 of the norm, zeros in x / in
// dy: 32 x 128->256 @56 at 50 / 85 %, 7.5 % of the products, 12.71 : 12.66, 0 / 93 %, 7 %, 13.01 : 13.04, 50 / 88 %, 6 %, 12.36 : 12.55, 77 / 77 %, 5.3 %,
// 12.40 : 12.48; 16 x 256->256 @56 at the same 13.16 : 13.09, 13.06 : 13.06, 12.85 : 13.03, 12.59 : 12.67)
constexpr long long kBwwHalfTiles = 48;

BwwArgs make_args(const st_conv_desc &d, int TH, int TW, bool tiles_over_input)
{
    BwwArgs A;
    A.sel = nullptr; A.want = 0; A.swapped = 0;
    A.N = d.N; A.C = d.C; A.K = d.K; A.H = d.H; A.W = d.W;
    A.OH = (d.H + 2 * d.pad_h - d.S) / d.stride_h + 1;
    A.OW = (d.W + 2 * d.pad_w - d.R) / d.stride_w + 1;
    A.pw = d.pad_w; A.ph = d.pad_h;
    const int eh = tiles_over_input ? d.H : A.OH, ew = tiles_over_input ? d.W : A.OW;
    A.tiles_h = ceil_div(eh, TH);
    A.tiles_w = ceil_div(ew, TW);
    const long long units = (long long)d.N * A.tiles_h * A.tiles_w;      // bounded by bww_fast_supported up to the tile size
    A.units = units < 0x7fffffffLL ? (int)units : 0x7fffffff;
    A.cgroups = ceil_div(d.C, 64);
    const int groups = ceil_div(d.K, 64) * A.cgroups;
    // number of partial sums: enough workgroups to fill the chip (256 compute units, 2 resident
    // workgroups each)
    int splits = ceil_div(kBwwTargetWorkgroups, groups);
    if (splits > A.units) splits = A.units;
    if (splits < 1) splits = 1;
    A.splits = splits;
    return A;
}

// tiles of the dense unit-stride 3x3 kernel: the shape that covers an image with fewer of them
bool dense_wide(const st_conv_desc &d)
{
    const int oh = d.H + 2 * d.pad_h - d.S + 1, ow = d.W + 2 * d.pad_w - d.R + 1;
    return (long long)ceil_div(oh, kDenseWideTH) * ceil_div(ow, kDenseWideTW) < (long long)ceil_div(oh, kDenseTH) * ceil_div(ow, kDenseTW);
}
BwwArgs dense_args(const st_conv_desc &d)
{
    BwwArgs A = bww_s2(d) ? make_args(d, kDenseS2TH, kDenseS2TW, false)
              : dense_wide(d) ? make_args(d, kDenseWideTH, kDenseWideTW, false) : make_args(d, kDenseTH, kDenseTW, false);
    // Two workgroups fit on a compute unit: not one more than that many (nine groups of 64 x 64 filters times 57 are 513, and
    // the last one took as long as the 512 before it; 320->320 @28, N = 8: 122 -> 89 us).
    const int groups = ceil_div(d.K, 64) * A.cgroups, resident = kBwwTargetWorkgroups / groups;
    if (resident >= 1 && A.splits > resident) A.splits = resident;
    // And no more than the workgroup with the most tiles calls for: with 512 for 784 tiles half of the workgroups take two
    // and the others write 18 MB of partial sums for nothing (64->64 @56, N = 8: 38 -> 35 us, 512->512 @14, N = 4: 48 -> 45).
    // Up to three tiles are left to one workgroup where the filters alone fill the chip: no partial sums and no launch to
    // add them up (one image, 512->512 @7: 22 -> 17).
    const int each = ceil_div(A.units, A.splits);
    A.splits = A.units <= 3 && groups >= 32 ? 1 : ceil_div(A.units, each);
    return A;
}

// Images whose offsets within four channel blocks, or whose sides, are too large for the 32 and 16 bits of BwwWideStage
bool bww_big_image(const BwwArgs &A)
{
    auto big = [](int H, int W) { return (long long)H * W >= 1 << 22 || H > 32000 || W > 32000; };
    return big(A.H, A.W) || big(A.OH, A.OW);
}

bool bww_half_tiles(const BwwArgs &A) { return A.units >= kBwwHalfTiles * A.splits && !bww_big_image(A); }

// Teams of a workgroup of the unit-stride kernel on bf16 pieces (BwwTeam).  The two share their barriers, which costs more than the partial gradients from
// some eight tiles on (one : two, us, tiles a team: 32 x 128->128 @28, 7, 58 : 54, 32 x 512->512 @14, 28, 148 : 150).  Where a group of 64 channels
// has at most 32, half of a team's wavefronts only stage, and two such teams on a
// compute unit leave it to others with two full ones (27 x 288->80 @39x8, 6, 41.3 : 43.0): up to two tiles only, and not where both channel counts end like
// that (3 x 80->48 @37x53 23.8 : 22.3, 20 x 48->32 @33x12 22.5 : 20.1, but 3 x 80->32 @54 20.2 : 23.1).
// The sum of two teams is rounded.  With hundreds of partial gradients the final sum of one for each team adds them up eight at a time in 32 bits, three
// roundings, and that of two all in 64 bits: together one (3 x 80->48 @37x53, 240 teams, 5.5e-8 -> 4.9e-8 of the norm).  With fewer than
// 120 few or none of them come in eights, and two teams would err more (2 x 256->256 @28, 32 teams, 5.0e-8 : 6.7e-8, though 36.8 : 31.0 us).
constexpr int kBwwTeamSplits = 120;
int bww_teams(const BwwArgs &A)
{
    if (A.splits < kBwwTeamSplits || A.splits * ceil_div(A.K, 64) * A.cgroups <= 256) return 1;
    const int tiles = ceil_div(A.units, A.splits);
    auto full = [](int channels) { return (channels + 63) % 64 >= 32; };
    if (tiles <= 2) return full(A.C) || full(A.K) ? 2 : 1;
    return full(A.C) && full(A.K) && tiles <= 8 ? 2 : 1;
}

template <int TH, int TW, int TEAMS>
void launch_bww_teams(const BwwArgs &A, const float *x, const float *dy, float *part, hipStream_t s)
{
    const dim3 grid(ceil_div(A.splits, TEAMS), ceil_div(A.K, 64) * A.cgroups), block(256 * TEAMS);
    if (bww_big_image(A)) hipLaunchKernelGGL((bww_dense_wide_kernel<3, 3, TH, TW, false, true, TEAMS>), grid, block, 0, s, A, x, dy, part);
    else hipLaunchKernelGGL((bww_dense_wide_kernel<3, 3, TH, TW, false, false, TEAMS>), grid, block, 0, s, A, x, dy, part);
}

template <int TH, int TW>
void launch_bww_dense_wide(const BwwArgs &A, const float *x, const float *dy, float *part, hipStream_t s)
{
    if (bww_half_tiles(A)) hipLaunchKernelGGL((bww_dense_half_kernel<TH, TW>), dim3(A.splits, ceil_div(A.K, 64) * A.cgroups), dim3(256), 0, s, A, x, dy, part);
    else if (A.units <= kBwwShortUnits && A.units <= 2 * A.splits && !bww_big_image(A))
        hipLaunchKernelGGL((bww_dense_wide_kernel<3, 3, TH, TW, true, false, 1>), dim3(A.splits, ceil_div(A.K, 64) * A.cgroups), dim3(256), 0, s, A, x, dy, part);
    else if (bww_teams(A) == 2) launch_bww_teams<TH, TW, 2>(A, x, dy, part, s);
    else launch_bww_teams<TH, TW, 1>(A, x, dy, part, s);
}

template <int TH, int TW, int PSTEP>
void launch_bww_dense_tiles(const BwwArgs &A, const float *x, const float *dy, float *part, hipStream_t s)
{
    const dim3 grid(A.splits, ceil_div(A.K, 64) * A.cgroups);
    if (A.units <= kBwwShortUnits && A.units <= 2 * A.splits)
        hipLaunchKernelGGL((bww_dense_kernel<3, 3, TH, TW, PSTEP, true>), grid, dim3(256), 0, s, A, x, dy, part);
    else hipLaunchKernelGGL((bww_dense_kernel<3, 3, TH, TW, PSTEP, false>), grid, dim3(256), 0, s, A, x, dy, part);
}

// partial gradients a launch of it writes (the workspace query counts one for each team)
int bww_dense_partials(const st_conv_desc &d, const BwwArgs &A) { return bww_s2(d) || bww_half_tiles(A) ? A.splits : ceil_div(A.splits, bww_teams(A)); }

// the 3x3 dense kernel with A = dense_args(d)
hipError_t launch_bww_dense_3x3(const st_conv_desc &d, const BwwArgs &A, const float *x, const float *dy, float *part, hipStream_t s)
{
    if (bww_s2(d)) launch_bww_dense_tiles<kDenseS2TH, kDenseS2TW, 2>(A, x, dy, part, s);
    else if (dense_wide(d)) launch_bww_dense_wide<kDenseWideTH, kDenseWideTW>(A, x, dy, part, s);
    else launch_bww_dense_wide<kDenseTH, kDenseTW>(A, x, dy, part, s);
    return hipGetLastError();
}

// tiles of the zero-skipping 3x3 kernel that tests the input of layer d
BwwArgs sparse_args(const st_conv_desc &d)
{
    return bww_s2(d) ? make_args(d, kSparseS2TH, kSparseS2TW, true) : make_args(d, kSparseTH, kSparseTW, true);
}

// 1x1 layers: chunks of kPwP pixels numbered across the minibatch; kw / cw = channels per workgroup
BwwArgs make_args_pw(const st_conv_desc &d, int kw, int cw, int chunk = kPwP, int target = kBwwTargetWorkgroups)
{
    BwwArgs A;
    A.sel = nullptr; A.want = 0; A.swapped = 0;
    A.N = d.N; A.C = d.C; A.K = d.K; A.H = d.H; A.W = d.W; A.OH = d.H; A.OW = d.W; A.pw = 0; A.ph = 0;
    A.tiles_h = A.tiles_w = 1;
    const long long chunks = ((long long)d.N * d.H * d.W + chunk - 1) / chunk;
    A.units = (int)chunks;                          // bww_fast_supported bounds N*H*W
    A.cgroups = ceil_div(d.C, cw);
    const int groups = ceil_div(d.K, kw) * A.cgroups;
    int splits = ceil_div(target, groups);
    if (splits > A.units) splits = A.units;
    if (splits < 1) splits = 1;
    A.splits = splits;
    return A;
}

// dense 1x1 BWW: channels of one operand per workgroup (128, or 64 for layers with no more than that), and the
// pixels per staged chunk that go with the tile
int pw_dense_tile(int channels) { return channels > 64 ? 128 : 64; }
constexpr int kPwDenseWorkgroups = 256;         // one of eight wavefronts per compute unit
template <int CW_, int KW_, int P_>
struct PwTile { static constexpr int CW = CW_, KW = KW_, P = P_; };
constexpr size_t pw_dense_lds(int cw, int kw, int p) { return (size_t)2 * 3 * (cw + kw) * p * 2; }
BwwArgs make_args_pw_dense(const st_conv_desc &d)
{
    const int cw = pw_dense_tile(d.C), kw = pw_dense_tile(d.K);
    // One workgroup fits on a compute unit: not one more than there are compute units (three groups of filters, 86 splits: 258
    // workgroups, of which the last two took as long as the 256 before them; 16->352 @200, N = 4: 127 -> 69 us, 512->1536 @7, N = 32: 43 -> 29)
    const int groups = ceil_div(d.K, kw) * ceil_div(d.C, cw), splits = kPwDenseWorkgroups / groups;
    return make_args_pw(d, kw, cw, cw == 128 && kw == 128 ? 32 : 64, groups * (splits > 1 ? splits : 1));
}

int pw_kpl(const st_conv_desc &d) { return d.K % 256 == 0 ? 4 : (d.K % 128 == 0 ? 2 : 1); }

size_t partial_bytes(const st_conv_desc &d, const BwwArgs &A)
{
    if (A.splits == 1) return 0;
    return (size_t)A.splits * d.K * d.C * d.S * d.R * sizeof(float);
}

hipError_t launch_reduce(const st_conv_desc &d, const Splits3 &sp, bool joined, const float *part, float *dw, const unsigned *sel, int want, hipStream_t s)
{
    const size_t n4 = (size_t)d.K * d.C * d.S * d.R / 4, nblk = (n4 + 63) / 64;
    const dim3 grid((unsigned)(nblk < kReduceGrid ? nblk : kReduceGrid));
    const float4 *p4 = reinterpret_cast<const float4 *>(part);
    float4 *dw4 = reinterpret_cast<float4 *>(dw);
    if (joined) hipLaunchKernelGGL(bww_reduce_kernel<true>, grid, dim3(1024), 0, s, p4, dw4, n4, sp, sel, want);
    else hipLaunchKernelGGL(bww_reduce_kernel<false>, grid, dim3(1024), 0, s, p4, dw4, n4, sp, sel, want);
    return hipGetLastError();
}

hipError_t reduce(const st_conv_desc &d, const BwwArgs &A, const float *part, float *dw, hipStream_t s, bool joined = false)
{
    if (A.splits == 1) return hipSuccess;               // the kernel wrote dw itself
    return launch_reduce(d, Splits3{{A.splits, A.splits, A.splits}}, joined, part, dw, A.sel, A.want, s);
}

}  // namespace

namespace {
bool bww_s2(const st_conv_desc &d)
{
    return d.stride_w == 2 && d.stride_h == 2 && d.R == 3 && d.S == 3 && d.pad_w == 1 && d.pad_h == 1;
}

// stride 2, dy tested: the tested tile runs over dy (OH x OW, K channels), the halo over x
BwwArgs make_args_s2_dy(const st_conv_desc &d)
{
    st_conv_desc e = d;
    e.C = d.K; e.K = d.C;
    e.H = (d.H + 2 * d.pad_h - d.S) / 2 + 1;
    e.W = (d.W + 2 * d.pad_w - d.R) / 2 + 1;
    e.stride_w = e.stride_h = 1;
    BwwArgs A = make_args(e, kS2TH, kS2TW, true);
    A.OH = d.H; A.OW = d.W;                         // size of the halo operand (x)
    A.pw = d.pad_w; A.ph = d.pad_h;
    return A;
}
}  // namespace

bool bww_fast_supported(const st_conv_desc &d)
{
    // gridDim.y carries (output-channel group, input-channel group), at least 32 channels each, with
    // either operand in either role
    if ((long long)ceil_div(d.K, 32) * ceil_div(d.C, 32) > 65535) return false;
    if (bww_s2(d)) return (long long)d.N * ceil_div(d.H, 4) * ceil_div(d.W, 8) <= 0x7fffffffLL;
    if (d.stride_w != 1 || d.stride_h != 1) return false;
    const long long units = (long long)d.N * ceil_div(d.H + 2 * d.pad_h, 7) * ceil_div(d.W + 2 * d.pad_w, 8);
    if (units > 0x7fffffffLL) return false;
    if (d.R == 3 && d.S == 3) return d.pad_w <= 2 && d.pad_h <= 2;
    if (d.R == 1 && d.S == 1)
        return d.pad_w == 0 && d.pad_h == 0 && (long long)d.N * d.H * d.W / kPwP < 0x7fffff00LL;
    return false;
}

size_t bww_sparse_workspace(const st_conv_desc &d)
{
    if (d.R == 1 && d.S == 1) return partial_bytes(d, make_args_pw(d, 64 * pw_kpl(d), 64));
    return partial_bytes(d, sparse_args(d));
}

bool bww_dense_half(const st_conv_desc &d)
{
    return d.R == 3 && d.stride_w == 1 && bww_fast_supported(d) && bww_half_tiles(dense_args(d));
}

size_t bww_dense_workspace(const st_conv_desc &d)
{
    if (d.R == 1 && d.S == 1) return partial_bytes(d, make_args_pw_dense(d));
    return partial_bytes(d, dense_args(d));
}

namespace {
// e = the layer as the kernel sees it (e.C tested channels, e.K lane channels); swapped = dy tested:
// the partial sums are then dw'[c][k] and go through the transposing reduction
hipError_t launch_pw_sparse(const st_conv_desc &d, const st_conv_desc &e, const float *tested, const float *other,
                            float *dw, float *ws, bool swapped, hipStream_t s, const unsigned *sel)
{
    const int kpl = pw_kpl(e);
    BwwArgs A = make_args_pw(e, 64 * kpl, 64);
    A.sel = sel; A.want = swapped ? 1 : 0; A.swapped = swapped ? 1 : 0;
    float *part = A.splits == 1 ? dw : ws;
    dim3 grid(A.splits, ceil_div(e.K, 64 * kpl) * A.cgroups);
    if (kpl == 4) hipLaunchKernelGGL(pw_bww_sparse_kernel<4>, grid, dim3(512), 0, s, A, tested, other, part);
    else if (kpl == 2) hipLaunchKernelGGL(pw_bww_sparse_kernel<2>, grid, dim3(512), 0, s, A, tested, other, part);
    else hipLaunchKernelGGL(pw_bww_sparse_kernel<1>, grid, dim3(512), 0, s, A, tested, other, part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return reduce(d, A, part, dw, s);
}
}  // namespace

// name of the kernel instance launch_bww_sparse runs for d (requires bww_fast_supported(d))
void bww_sparse_kernel_name(const st_conv_desc &d, char *buf, size_t len)
{
    if (bww_direct(d)) snprintf(buf, len, "bww_direct_kernel<%d>", d.R);
    else if (d.R == 1) snprintf(buf, len, "pw_bww_sparse_kernel<%d>", pw_kpl(d));
    else if (bww_s2(d)) snprintf(buf, len, "bww_sparse_kernel<3, 3, %d, %d, 1>", kSparseS2TH, kSparseS2TW);
    else snprintf(buf, len, "bww_sparse_kernel<3, 3, %d, %d, 0>", kSparseTH, kSparseTW);
}

hipError_t launch_bww_sparse(const st_conv_desc &d, const float *x, const float *dy, float *dw,
                             float *ws, hipStream_t s, const unsigned *sel)
{
    if (!sel && bww_direct(d)) return launch_bww_direct(d, x, dy, dw, 0, nullptr, s);
    if (d.R == 1) return launch_pw_sparse(d, d, x, dy, dw, ws, false, s, sel);
    BwwArgs A = sparse_args(d);
    A.sel = sel; A.want = 0;
    float *part = A.splits == 1 ? dw : ws;
    dim3 grid(A.splits, ceil_div(d.K, 64) * A.cgroups);
    if (bww_s2(d)) {
        hipLaunchKernelGGL((bww_sparse_kernel<3, 3, kSparseS2TH, kSparseS2TW, 1>), grid, dim3(512), 0, s, A, x, dy, part);
        hipError_t err = hipGetLastError();
        return err != hipSuccess ? err : reduce(d, A, part, dw, s);
    }
    hipError_t e = allow_dynamic_lds<bww_sparse_kernel<3, 3, kSparseTH, kSparseTW, 0>>(kSparseLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bww_sparse_kernel<3, 3, kSparseTH, kSparseTW, 0>), grid, dim3(512), kSparseLds, s, A, x, dy, part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce(d, A, part, dw, s);
}

// BWW that tests dy: the same kernel with the operand roles exchanged.  With unit stride,
//   dw[k,c,v,u] = sum x[n,c,oh-ph+v,ow-pw+u] dy[n,k,oh,ow] = sum dy[n,k,ih-ph'+v',iw-pw'+u'] x[n,c,ih,iw]
// for v' = S-1-v, ph' = S-1-ph (same for the width), i.e. the filter gradient of a layer whose
// input is dy (K channels, OH x OW, padding S-1-pad) and whose output gradient is x (C channels).
namespace {
st_conv_desc swapped_desc(const st_conv_desc &d)
{
    st_conv_desc e = d;
    e.C = d.K; e.K = d.C;
    e.H = d.H + 2 * d.pad_h - d.S + 1;
    e.W = d.W + 2 * d.pad_w - d.R + 1;
    e.pad_h = d.S - 1 - d.pad_h;
    e.pad_w = d.R - 1 - d.pad_w;
    return e;
}
}  // namespace

bool bww_dy_fast_supported(const st_conv_desc &d)
{
    if (bww_s2(d)) return bww_fast_supported(d);
    return bww_fast_supported(d) && d.pad_h <= d.S - 1 && d.pad_w <= d.R - 1 && bww_fast_supported(swapped_desc(d));
}

size_t bww_sparse_dy_workspace(const st_conv_desc &d)
{
    if (d.R == 1 && d.S == 1) {
        const st_conv_desc e = swapped_desc(d);
        return (size_t)make_args_pw(e, 64 * pw_kpl(e), 64).splits * d.K * d.C * sizeof(float);
    }
    if (bww_s2(d)) return (size_t)make_args_s2_dy(d).splits * d.K * d.C * d.S * d.R * sizeof(float);
    const st_conv_desc e = swapped_desc(d);
    const BwwArgs A = make_args(e, kSparseTH, kSparseTW, true);
    return (size_t)A.splits * d.K * d.C * d.S * d.R * sizeof(float);
}

hipError_t launch_bww_sparse_dy(const st_conv_desc &d, const float *x, const float *dy, float *dw,
                                float *ws, hipStream_t s, const unsigned *sel)
{
    if (!sel && bww_direct(d)) return launch_bww_direct(d, x, dy, dw, 1, nullptr, s);
    if (bww_s2(d)) {
        BwwArgs A = make_args_s2_dy(d);
        A.sel = sel; A.want = 1; A.swapped = 1;
        float *part = A.splits == 1 ? dw : ws;
        dim3 grid(A.splits, ceil_div(A.K, 64) * A.cgroups);
        hipLaunchKernelGGL((bww_sparse_kernel<3, 3, kS2TH, kS2TW, 2>), grid, dim3(512), 0, s, A, dy, x, part);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        return reduce(d, A, part, dw, s);
    }
    const st_conv_desc e = swapped_desc(d);
    if (d.R == 1) return launch_pw_sparse(d, e, dy, x, dw, ws, true, s, sel);
    BwwArgs A = make_args(e, kSparseTH, kSparseTW, true);
    A.sel = sel; A.want = 1; A.swapped = 1;
    float *part = A.splits == 1 ? dw : ws;
    dim3 grid(A.splits, ceil_div(e.K, 64) * A.cgroups);
    hipError_t err = allow_dynamic_lds<bww_sparse_kernel<3, 3, kSparseTH, kSparseTW, 0>>(kSparseLds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL((bww_sparse_kernel<3, 3, kSparseTH, kSparseTW, 0>), grid, dim3(512), kSparseLds, s, A, dy, x, part);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    return reduce(d, A, part, dw, s);
}

// st_conv_bww_auto on unit-stride 3x3 layers: one zero-skipping launch that carries the arguments of both
// operand roles and computes the selected one, the dense launch, and one launch that adds up the partial
// sums of whichever form ran.  All three forms stage their partial sums in ws (also a single one).
bool bww_auto_merged_supported(const st_conv_desc &d)
{
    return d.R == 3 && d.S == 3 && d.stride_w == 1 && d.stride_h == 1 && bww_fast_supported(d) && bww_dy_fast_supported(d);
}

hipError_t launch_bww_auto_merged(const st_conv_desc &d, const float *x, const float *dy, float *dw, float *ws,
                                  hipStream_t s, const unsigned *sel)
{
    const st_conv_desc e = swapped_desc(d);
    BwwArgs A0 = make_args(d, kSparseTH, kSparseTW, true), A1 = make_args(e, kSparseTH, kSparseTW, true);
    BwwArgs A2 = dense_args(d);
    A0.sel = A1.sel = A2.sel = sel;
    A0.want = kEitherOperand; A1.want = kEitherOperand; A1.swapped = 1; A2.want = 2;
    const bool direct = bww_direct(d);                              // small layers: writes dw itself
    hipError_t err;
    if (direct) {
        if ((err = launch_bww_direct(d, x, dy, dw, 0, sel, s)) != hipSuccess) return err;
    } else {
        const int ygroups = ceil_div(d.K, 64) * ceil_div(d.C, 64);  // the same for both operand roles
        dim3 grid(A0.splits > A1.splits ? A0.splits : A1.splits, ygroups);
        err = allow_dynamic_lds<bww_sparse_either_kernel<3, 3, kSparseTH, kSparseTW>>(kSparseLds);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((bww_sparse_either_kernel<3, 3, kSparseTH, kSparseTW>), grid, dim3(512), kSparseLds, s, A0, A1, x, dy, ws);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    if ((err = launch_bww_dense_3x3(d, A2, x, dy, ws, s)) != hipSuccess) return err;
    const int partials = bww_dense_partials(d, A2);
    return launch_reduce(d, Splits3{{A0.splits, A1.splits, partials}}, partials < A2.splits, ws, dw, sel, direct ? 2 : kAnyForm, s);
}

hipError_t launch_bww_dense(const st_conv_desc &d, const float *x, const float *dy, float *dw,
                            float *ws, hipStream_t s, const unsigned *sel)
{
    if (d.R == 1) {
        BwwArgs A1 = make_args_pw_dense(d);
        A1.sel = sel; A1.want = 2;
        const int cw = pw_dense_tile(d.C), kw = pw_dense_tile(d.K);
        dim3 grid1(A1.splits, ceil_div(d.K, kw) * A1.cgroups);
        float *part1 = A1.splits == 1 ? dw : ws;
        auto launch = [&](auto cfg) {
            using C = decltype(cfg);
            constexpr auto kern = pw_bww_dense_kernel<C::CW, C::KW, C::P>;
            constexpr size_t lds = pw_dense_lds(C::CW, C::KW, C::P);
            const hipError_t e = allow_dynamic_lds<kern>(lds);
            if (e == hipSuccess) hipLaunchKernelGGL(kern, grid1, dim3(512), lds, s, A1, x, dy, part1);
            return e;
        };
        hipError_t err = cw == 128 ? (kw == 128 ? launch(PwTile<128, 128, 32>{}) : launch(PwTile<128, 64, 64>{}))
                                   : (kw == 128 ? launch(PwTile<64, 128, 64>{}) : launch(PwTile<64, 64, 64>{}));
        if (err != hipSuccess) return err;
        err = hipGetLastError();
        return err != hipSuccess ? err : reduce(d, A1, ws, dw, s);
    }
    BwwArgs A = dense_args(d);
    A.sel = sel; A.want = 2;
    const int partials = bww_dense_partials(d, A);
    float *part = partials == 1 ? dw : ws;
    hipError_t e = launch_bww_dense_3x3(d, A, x, dy, part, s);
    if (e != hipSuccess) return e;
    const bool joined = partials < A.splits;
    A.splits = partials;
    return reduce(d, A, part, dw, s, joined);
}

// The 3x3 zero-skipping forms pass the dense one between 95 and 99 % zeros (N = 32, us, both with all launches of the entry point, zero-skipping at
// 80 / 95 / 99 % : dense: 256->256 @56 667 / 507 / 292 : 461, @28 193 / 154 / 100 : 157, 64->64 @112 191 / 151 / 108 : 141; few channels, whose lanes
// they do not fill, 16->32 @112 156 / 107 / 69 : 94, 9 x 16->176 @181 551 at 80 % : 252; 4 x 64->128 @24 30.8 / 27.5 / 24.6 : 25.8): 96 %, as far as
// enough products are not zero (kSelThrFew).  Launches of less than 128 million multiply-adds keep the line of 75 %, from which on callers of this entry
// point have always had the sparser operand tested (2 x 64->128 @24 at 80 % 27.4 : 22).  So do those whose zero-skipping partial gradients come from three tiles or
// fewer and, neither eight of them nor 120 and more, are not added up eight at a time in 32 bits: with few products a sum they err less than the dense
// form's of more than one tile (zero-skipping : dense, 77 % zeros in both, 1e-8 of the norm, us: 2 x 256->256 @28 4.61 : 4.82, 47 : 42, 6 x 128->128 @28 4.63 : 4.93, 42 : 36, 8 x 128->256 @28
// 5.35 : 5.64, 56 : 51, 12 x 128->256 @28 6.10 : 6.26, 68 : 59; not 8 x 256->256 @28, four tiles, 6.63 : 6.35, 4 x 512->512 @14, eight gradients, 6.59 : 5.49,
// 4 x 128->128 @40, 120 of them, 5.76 : 4.81, 4 x 64->128 @24, a tile each in the dense form too, 4.59 : 4.17).
// Launches of at most 128 tiles that give every workgroup one of them and write 24 MB of partial gradients or more are bound by
// these, and the dense form's smaller tiles leave more of them (zero-skipping at 30 / 50 / 70 % zeros : dense: 208->256 @9
// N = 4 26.6 / 25.8 / 24.8 : 30.8, 512->256 @10 N = 2 29.4 / 28.9 / 28.4 : 32.8, 256->256 @28 N = 1 32.9 / 32.0 / 31.1 : 36.3, 336->192
// @12 N = 2 24.0 / 23.2 / 22.3 : 25.9; with less, 64->128 @14 N = 4 23.1 / 22.3 / 21.4 : 17.0, or more tiles, 64->64 @56 N = 2 29.8 /
// 28.9 / 28.0 : 26.1, 80->48 @37x53 N = 3 at 50 % 29.4 : 25.5): from 25 % on.
// A 1x1 layer saves at most K/64 (or C/64) multiply-adds per zero and stays behind the matrix cores at every zero
// fraction measured (up to 95 %): never (1001).  (Stride-2 layers never get here: they are decided by size, unsampled.)
unsigned bww_sparse_threshold(const st_conv_desc &d)
{
    if (!bww_fast_supported(d)) return 0;           // generic kernels: the test only ever removes work
    if (d.R == 1) return 1001;
    const BwwArgs A = dense_args(d);
    const long long partial_bytes = (long long)A.units * d.K * d.C * (9 * (int)sizeof(float));
    if (A.splits == A.units && A.units <= 128 && partial_bytes >= 24000000) return 250;
    const BwwArgs Z = make_args(d, kSparseTH, kSparseTW, true);
    const bool exact_sums = Z.units <= 3 * Z.splits && Z.splits > 8 && Z.splits < kBwwTeamSplits && A.units > A.splits;
    return !exact_sums && (double)d.N * A.OH * A.OW * d.C * d.K * 9. >= 128e6 ? 960 : 750;
}

}  // namespace st
