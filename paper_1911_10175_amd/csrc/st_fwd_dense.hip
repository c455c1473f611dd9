// Dense correlation on the matrix cores, 3x3 at stride 1 and 2: the form without tests the zero-skipping kernels are
// measured against (the role the library's dense "direct" convolution plays in SparseTrain
// Sec. 4).  Used for FWD and, with transposed filters, for BWI.
//
// Implicit GEMM with v_mfma_f32_32x32x16_bf16 on the bf16 pieces of both operands (st_split.hpp): rows = 32 output
// channels, columns = 32 output pixels, reduction = the 16 input channels of a block for one filter tap, six
// instructions per tap and block.  A wavefront owns an 8x8 (4x14, 2x28) pixel tile times 32 output channels (two
// accumulator blocks).  The 4 wavefronts of a workgroup cover KQ column blocks of 4/KQ pixel tiles; the wavefronts
// that share a pixel tile stage its input halo for one 16-channel block cooperatively in LDS, split into pieces on
// the way (zero padding is applied there once), double-buffered: the global loads for block cb+1 are issued at
// the first tap of block cb and written to the other buffer after the last tap, one barrier per block.  For every
// tap the input operand is read from LDS at the shifted pixel.  The filters come from
// a copy that a small prologue kernel writes into the workspace, already split, in the order the MFMA lanes
// consume it, [K/32][C/16][tap][piece][c half][32 k][8 c].  No tests, no skipping.
//
// Measured (N = 32; the same structure on v_mfma_f32_32x32x2_f32 -> now): 256->256 @56 1022 -> 555 us (213 TFLOP/s;
// the bare instruction stream reaches 1800 / 6 = 300), 512->512 @28 1090 -> 613, 512->512 @14 292 -> 182,
// 128->128 @28 78 -> 49, 512->512 @7 92 -> 67, 128->128 @56 stride 2 86 -> 52.  Counters on 256->256 @56: matrix pipe
// busy 65 % of the time (3136 workgroups are 3.06 rounds of the 1024 resident ones), LDS 50 %, two thirds of it bank
// conflicts where a tile row ends.
#include <cstdlib>

#include "st_common.hpp"
#include "st_filter_copies.hpp"
#include "st_fwd_dense_impl.hpp"

namespace st {
namespace {

// Prologue: filters in MFMA consumption order (st_filter_copies.hpp).
__global__ __launch_bounds__(256) void reformat_filters_kernel(int Ko, int Ci, int S, int R, int transpose,
                                                               const float *__restrict__ w,
                                                               float *__restrict__ wd, size_t total,
                                                               const unsigned *sel, unsigned thr)
{
    if (form_deselected(sel, 1, thr)) return;       // the copy of a form that will not run is not written
    reformat_filters_block(blockIdx.x, Ko, Ci, S, R, transpose, w, wd, total);
}

__global__ __launch_bounds__(256) void pw_filters_kernel(int Ko, int Ci, int transpose, const float *__restrict__ w,
                                                         float *__restrict__ wd, size_t total, const unsigned *sel, unsigned thr)
{
    if (form_deselected(sel, 1, thr)) return;
    pw_filters_block(blockIdx.x, Ko, Ci, transpose, w, wd, total);
}

// 1x1 layers served by the pixel-wise kernel (st_pw_dense.hip); its minibatch-wide pixel numbers are kept in int
bool pointwise(const Geom &g) { return g.R == 1 && g.S == 1 && (long long)g.N * g.Ho * g.Wo <= 0x7fffff00LL; }

// out += part[0] + part[1] + ... (splits - 1 of them, in that order), float4 at a time, on a capped grid
__global__ __launch_bounds__(256) void sum_partials_kernel(const float4 *__restrict__ part, float4 *__restrict__ out,
                                                           size_t n4, int splits, const unsigned *sel, unsigned thr)
{
    if (form_deselected(sel, 1, thr)) return;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
        float4 a = out[i];
        for (int p = 1; p < splits; ++p) {
            const float4 v = part[(size_t)(p - 1) * n4 + i];
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
        out[i] = a;
    }
}

template <int R, int S, int KQ, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
hipError_t launch_cfg(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    using Cfg = FwdDenseCfg<R, S, TWD, MODE, PI, PJ>;
    constexpr int TQ = 4 / KQ;
    // MODE 2 tiles the positions of one parity class: (Ho - PI + 1) / 2 rows, (Wo - PJ + 1) / 2 columns
    const int rows = MODE == 2 ? (g.Ho - PI + 1) / 2 : g.Ho, cols = MODE == 2 ? (g.Wo - PJ + 1) / 2 : g.Wo;
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int tiles_w = ceil_div(cols, Cfg::TW), tiles_h = ceil_div(rows, Cfg::TH);
    const long long total_tiles = (long long)tiles_w * tiles_h * g.N;
    const int kgroups = ceil_div(g.Ko, 32 * KQ);
    const long long blocks = (total_tiles + TQ - 1) / TQ * kgroups;
    if (total_tiles > 0x7fffffffLL || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const int cs = MODE == 0 ? dense_channel_split(g) : 1;
    const size_t n_out = (size_t)g.N * g.Ko * g.Ho * g.Wo;
    // partial outputs of the shares after the first sit behind the filter copy in the workspace
    float *part = cs > 1 ? const_cast<float *>(wd) + (fwd_dense_filter_bytes(g) + 255) / 256 * 256 / sizeof(float) : nullptr;
    hipLaunchKernelGGL((fwd_dense_kernel<R, S, KQ, TWD, MODE, PI, PJ>), dim3((unsigned)blocks, cs), dim3(256), 0, s, g, in, wd,
                       out, part, tiles_w, tiles_h, kgroups, (int)total_tiles, cs, n_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || cs == 1) return e;
    const size_t n4 = n_out / 4;
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)(n4 / 256 + 1 < 1024 ? n4 / 256 + 1 : 1024)), dim3(256), 0, s,
                       reinterpret_cast<const float4 *>(part), reinterpret_cast<float4 *>(out), n4, cs, g.sel, g.thr);
    return hipGetLastError();
}

template <int R, int S, int TWD, int MODE = 0, int PI = 0, int PJ = 0>
hipError_t launch_kq(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    // the stride-2 halo is four times larger: one pixel tile per workgroup is all that fits in LDS
    // (with at most 64 output channels some of its four wavefronts then only help staging)
    if constexpr (MODE == 1) {
        return launch_cfg<R, S, 4, TWD, MODE, PI, PJ>(g, in, wd, out, s);
    } else {
        if (g.Ko > 64) return launch_cfg<R, S, 4, TWD, MODE, PI, PJ>(g, in, wd, out, s);
        if (g.Ko > 32) return launch_cfg<R, S, 2, TWD, MODE, PI, PJ>(g, in, wd, out, s);
        return launch_cfg<R, S, 1, TWD, MODE, PI, PJ>(g, in, wd, out, s);
    }
}

// stride-2 FWD: 8x8 output tiles (17x17 input halo), 4x14 tiles (9x29) for 14-wide outputs
hipError_t launch_s2_fwd(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    if (g.Wo % 8 != 0 && g.Wo % 14 == 0 && g.Ho % 4 <= g.Ho % 8) return launch_kq<3, 3, 14, 1>(g, in, wd, out, s);
    return launch_kq<3, 3, 8, 1>(g, in, wd, out, s);
}

// BWI of a stride-2 layer: the four parity classes of the dx positions in one launch, the longest (4 taps) first.  As
// four launches of a quarter of the workgroups each they left most of the chip idle (N = 32, us: 128->128 @56 77 -> 58,
// 256->256 @28 114 -> 63, 512->512 @14 194 -> 91).
struct ParityGrid {
    int tiles_w[4], tiles_h[4], total_tiles[4];     // of class 3 - 2*PI - PJ
    unsigned first[5];                              // first workgroup of each class
};

template <int KQ, int TWD>
__global__ __launch_bounds__(256, (FwdDenseCfg<3, 3, TWD, 2, 1, 1>::minw(KQ))) void fwd_dense_s2_bwi_kernel(
    Geom g, const float *__restrict__ in, const float *__restrict__ wd, float *__restrict__ out, ParityGrid q, int kgroups)
{
    if (form_deselected(g.sel, g.want, g.thr)) return;
    __shared__ __attribute__((aligned(16))) float lds_all[fwd_dense_lds_floats<3, 3, KQ, TWD, 2, 1, 1>()];     // the largest of the four
    static_for<0, 4>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value, PI = (3 - i) / 2, PJ = (3 - i) % 2;
        if (blockIdx.x >= q.first[i] && blockIdx.x < q.first[i + 1])            // uniform over the workgroup
            fwd_dense_body<3, 3, KQ, TWD, 2, PI, PJ>(g, in, wd, out, nullptr, q.tiles_w[i], q.tiles_h[i], kgroups, q.total_tiles[i], 1, 0,
                                                     (int)(blockIdx.x - q.first[i]), 0, lds_all);
    });
}

template <int KQ, int TWD>
hipError_t launch_s2_bwi_kq(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    constexpr int TQ = 4 / KQ, TH = 64 / TWD;
    ParityGrid q;
    const int kgroups = ceil_div(g.Ko, 32 * KQ);
    long long blocks = 0;
    for (int i = 0; i < 4; ++i) {
        const int PI = (3 - i) / 2, PJ = (3 - i) % 2;
        q.tiles_w[i] = ceil_div((g.Wo - PJ + 1) / 2, TWD);
        q.tiles_h[i] = ceil_div((g.Ho - PI + 1) / 2, TH);
        const long long tiles = (long long)q.tiles_w[i] * q.tiles_h[i] * g.N;
        if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
        q.total_tiles[i] = (int)tiles;
        q.first[i] = (unsigned)blocks;
        blocks += (tiles + TQ - 1) / TQ * kgroups;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    }
    q.first[4] = (unsigned)blocks;
    hipLaunchKernelGGL((fwd_dense_s2_bwi_kernel<KQ, TWD>), dim3((unsigned)blocks), dim3(256), 0, s, g, in, wd, out, q, kgroups);
    return hipGetLastError();
}

template <int TWD>
hipError_t launch_s2_bwi_tw(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    if (g.Ko > 64) return launch_s2_bwi_kq<4, TWD>(g, in, wd, out, s);
    if (g.Ko > 32) return launch_s2_bwi_kq<2, TWD>(g, in, wd, out, s);
    return launch_s2_bwi_kq<1, TWD>(g, in, wd, out, s);
}

hipError_t launch_s2_bwi(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    const int cols = g.Wo / 2;                      // columns of a parity class (up to one more for PJ = 0)
    if (cols % 8 != 0 && cols % 14 == 0) return launch_s2_bwi_tw<14>(g, in, wd, out, s);
    return launch_s2_bwi_tw<8>(g, in, wd, out, s);
}

template <int R, int S>
hipError_t launch_rs(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    int twd, kq;
    long long blocks;
    dense_tiling(g, &twd, &kq, &blocks);
    if (twd == 28) return launch_kq<R, S, 28>(g, in, wd, out, s);
    if (twd == 14) return launch_kq<R, S, 14>(g, in, wd, out, s);
    return launch_kq<R, S, 8>(g, in, wd, out, s);
}

}  // namespace

bool fwd_dense_supported(const Geom &g)
{
    if (g.sw != g.sh || g.uw != g.uh) return false;
    if (g.sw == 2 && g.uw == 1) return g.R == 3 && g.S == 3 && g.pw <= 2 && g.ph <= 2;
    if (g.sw == 1 && g.uw == 2) return g.R == 3 && g.S == 3 && g.pw == 1 && g.ph == 1;
    if (g.sw != 1 || g.uw != 1) return false;
    if (g.R == 3 && g.S == 3) return g.pw <= 2 && g.ph <= 2;
    if (g.R == 1 && g.S == 1) return g.pw == 0 && g.ph == 0;
    return false;
}

size_t fwd_dense_filter_bytes(const Geom &g)
{
    // output channels padded to a multiple of 128 so that every column block a workgroup touches exists
    // (three bf16 pieces per element; the pixel-wise 1x1 kernel takes fp32)
    return (size_t)ceil_div(g.Ko, 128) * 128 * g.Ci * g.S * g.R * (pointwise(g) ? 4 : 6);
}

size_t fwd_dense_workspace_bytes(const Geom &g)
{
    // filter copy, then the partial outputs of a channel-split launch
    // (the first share writes the output itself)
    const size_t n = fwd_dense_filter_bytes(g), out = (size_t)g.N * g.Ko * g.Ho * g.Wo * sizeof(float);
    const int cs = dense_channel_split(g);
    if (cs == 1) return n;
    const size_t need = (n + 255) / 256 * 256 + (size_t)(cs - 1) * out;
    // never less than the fp32 copy and the partial outputs this query has always counted for such a launch
    const size_t before = (n / 6 * 4 + 255) / 256 * 256 + (size_t)dense_channel_split_pow2(g) * out;
    return need > before ? need : before;
}

hipError_t launch_reformat_filters(const Geom &g, bool transpose, const float *w, float *wd, hipStream_t s)
{
    if (pointwise(g)) {
        const size_t n = fwd_dense_filter_bytes(g) / 4;
        hipLaunchKernelGGL(pw_filters_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g.Ko, g.Ci, transpose ? 1 : 0, w, wd, n,
                           g.sel, g.thr);
        return hipGetLastError();
    }
    const size_t total = fwd_dense_filter_bytes(g) / 48;                 // 8 elements per thread
    hipLaunchKernelGGL(reformat_filters_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, g.Ko, g.Ci,
                       g.S, g.R, transpose ? 1 : 0, w, wd, total, g.sel, g.thr);
    return hipGetLastError();
}

hipError_t launch_fwd_dense(const Geom &g, const float *in, const float *wd, float *out, hipStream_t s)
{
    if (g.sw == 2) return launch_s2_fwd(g, in, wd, out, s);
    if (g.uw == 2) return launch_s2_bwi(g, in, wd, out, s);
    if (g.R == 3 && g.S == 3) return launch_rs<3, 3>(g, in, wd, out, s);
    if (g.R == 1 && g.S == 1) return pointwise(g) ? launch_pw_dense(g, in, wd, out, s) : launch_rs<1, 1>(g, in, wd, out, s);
    return hipErrorInvalidValue;
}

}  // namespace st
