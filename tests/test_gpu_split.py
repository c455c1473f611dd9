"""The dense kernels form fp32 products from bf16 pieces on the matrix cores: fp32 accuracy on ordinary values, and
plain fp32 results where a value lies outside the range of the pieces.  Every test here needs an MI355X."""
import numpy as np
import pytest
import torch

import stgen
from oracle import st_ref
from oracle.st_ref import Geom

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1911_10175_amd as st
    from tests.gpu_harness import DeviceLayer, desc_of
    from tests.kernel_choice import dense_kernel

# one geometry per kernel shape: column blocks per workgroup (16 / 48 / 80 and more produced channels), strips of unequal
# widths, tiles that span many images or are cut short by their halo, the channel split, stride 2 (and its four parity
# classes in BWI), 1x1
GEOMS = {
    "3x3 16->48": Geom(2, 16, 48, 9, 11, 3, 3, 1, 1, 1, 1),
    "3x3 80->144": Geom(2, 80, 144, 7, 28, 3, 3, 1, 1, 1, 1),
    "3x3 48->32 pad2": Geom(1, 48, 32, 5, 12, 3, 3, 1, 1, 2, 2),
    "3x3 split": Geom(1, 256, 256, 7, 7, 3, 3, 1, 1, 1, 1),
    "3x3 stride 2": Geom(2, 48, 80, 13, 10, 3, 3, 2, 2, 1, 1),
    "3x3 tiny images": Geom(70, 16, 144, 2, 3, 3, 3, 1, 1, 1, 1),
    "3x3 one row": Geom(5, 16, 32, 1, 230, 3, 3, 1, 1, 1, 1),
    "3x3 stride 2 tiny images": Geom(40, 32, 16, 3, 4, 3, 3, 2, 2, 1, 1),
    "3x3 stride 2 16->80": Geom(2, 16, 80, 9, 12, 3, 3, 2, 2, 1, 1),
    "1x1 64->64": Geom(3, 64, 64, 53, 53, 1, 1),
    "1x1 80->48": Geom(2, 80, 48, 5, 7, 1, 1),
    # enough pixels for the 1x1 kernel on pieces: 1, 2 and 4 column blocks per workgroup, short and long reductions
    "1x1 64->32": Geom(8, 64, 32, 65, 64, 1, 1),
    "1x1 32->48": Geom(8, 32, 48, 64, 65, 1, 1),
    "1x1 144->80": Geom(4, 144, 80, 65, 64, 1, 1),
}


def inputs(g, seed):
    x = stgen.relu_sparse(g.x_shape, 0.5, 4 * seed)
    w = stgen.he_normal(g.w_shape, 4 * seed + 1)
    dy = stgen.bernoulli_masked(g.y_shape, 0.5, 4 * seed + 2, 4 * seed + 3)
    return x, w, dy


def refs(g, x, w, dy):
    return {"fwd": st_ref.conv_fwd(g, x, w), "bwi": st_ref.conv_bwi(g, dy, w), "bww": st_ref.conv_bww(g, x, dy)}


def terms(g):
    """Products per output.  An fp32 sum of n products in any order is within (n + 1) 2^-24 of the sum of their
    magnitudes, the pieces left out of a product are within 2^-23 of it, and n results below the smallest normal number
    may each be off by half the smallest subnormal."""
    return {"fwd": g.C * g.R * g.S, "bwi": g.K * g.R * g.S, "bww": g.N * g.OH * g.OW}


def check(g, x, w, dy, label):
    L = DeviceLayer(g, x, w, dy)
    for p, (ref, ref_abs) in refs(g, x, w, dy).items():
        got = getattr(L, p)(True).astype(np.float64)
        n = terms(g)[p]
        fine = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), f"{label} {p}: NaN elsewhere"
        inf = np.isinf(ref)
        assert np.array_equal(got[inf], ref[inf]), f"{label} {p}: infinities"
        off = np.abs(got[fine] - ref[fine])
        bound = (n + 3) * 2.0 ** -24 * ref_abs[fine] + n * 2.0 ** -150
        assert np.all(off <= bound), f"{label} {p}: {np.max(off / np.maximum(bound, 1e-300))} of the bound"


@pytest.mark.parametrize("name", GEOMS)
def test_dense_forms_keep_fp32_accuracy(name):
    """Values of very different size side by side, each output within the bound of an fp32 sum.  (The bound grows with the number
    of terms, so a lost third piece need not break it: test_short_reductions_err_no_more_than_fp32_instructions sees that.)"""
    g = GEOMS[name]
    x, w, dy = inputs(g, 11)
    rng = np.random.default_rng(5)
    for t in (x, w, dy):
        t *= np.float32(2.0) ** rng.integers(-20, 21, t.shape).astype(np.float32)
    check(g, x, w, dy, name)


@pytest.mark.parametrize("name", GEOMS)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, 1e-30, 1e-35, 1e-42])
def test_dense_forms_outside_the_range_of_the_pieces(name, value):
    """Infinities, NaN, the largest and the smallest values: in x, in dy and in w, a few elements each."""
    g = GEOMS[name]
    for where in range(3):
        x, w, dy = inputs(g, 13)
        # no zeros in the other tensors (0 * inf: the padding's share is not defined) and no overflow of finite sums
        for t in (x, w, dy):
            t[t == 0] = 0.25
            t *= 2.0 ** -6
        t = (x, w, dy)[where].reshape(-1)
        t[[0, t.size // 3, t.size - 1]] = value
        check(g, x, w, dy, f"{name} {value} in {'x w dy'.split()[where]}")


def test_dense_forms_on_subnormal_tensors():
    """A whole tensor below the smallest normal number against huge filters."""
    g = GEOMS["3x3 16->48"]
    x, w, dy = inputs(g, 17)
    check(g, x * np.float32(1e-39), w * np.float32(1e34), dy * np.float32(1e-39), "subnormal")


@pytest.mark.parametrize("p,dense", [(0.5, True), (0.8, True), (0.99, False)])
@pytest.mark.parametrize("name", ["fwd", "bwi"])
def test_auto_switches_late_with_128_reduced_channels(name, p, dense):
    """The self-selecting entry points, one main kernel for both forms: bit for bit the form the zero fraction asks for."""
    g = Geom(8, 128, 128, 56, 56, 3, 3, 1, 1, 1, 1)
    x = stgen.relu_sparse(g.x_shape, p, 4)
    w = stgen.he_normal(g.w_shape, 5)
    dy = stgen.bernoulli_masked(g.y_shape, p, 6, 7)
    L = DeviceLayer(g, x, w, dy)
    run = getattr(L, name)
    got = run("auto", raw=True)
    assert torch.equal(got, run(dense, raw=True))
    assert not torch.equal(got, run(not dense, raw=True)), "forms indistinguishable: test is void"


def test_dense_forms_on_products_near_the_smallest_normal_number():
    """Factors in the normal range whose products, and the products of their pieces, are not."""
    for name in ("3x3 80->144", "3x3 stride 2", "1x1 64->64"):
        g = GEOMS[name]
        x, w, dy = inputs(g, 19)
        check(g, x * np.float32(2.0 ** -62), w * np.float32(2.0 ** -62), dy * np.float32(2.0 ** -64), name)
        check(g, x * np.float32(2.0 ** -118), w, dy * np.float32(2.0 ** -118), name)


def as_products(g, x, w, dy, name):
    """The pass as a matrix product [rows][terms] x [terms][columns] and the function that brings a plain result of the
    pass into that shape."""
    xt, wt, dyt = (torch.from_numpy(t).double() for t in (x, w, dy))        # (fwd does not look at dy, nor bwi at x)
    unfold = torch.nn.functional.unfold
    if name == "fwd":
        cols = unfold(xt, (g.S, g.R), padding=(g.pad_h, g.pad_w), stride=(g.stride_h, g.stride_w))          # [N][C S R][OH OW]
        return wt.reshape(g.K, -1), cols.transpose(0, 1).reshape(cols.shape[1], -1), lambda y: y.transpose(1, 0, 2, 3).reshape(g.K, -1)
    if name == "bwi":                                   # dy spread out by the stride, filters transposed and reversed
        H, W = g.H + 2 * g.pad_h - g.S + 1, g.W + 2 * g.pad_w - g.R + 1
        spread = torch.zeros((g.N, g.K, H, W), dtype=torch.float64)
        spread[:, :, ::g.stride_h, ::g.stride_w] = dyt[:, :, :(H + g.stride_h - 1) // g.stride_h, :(W + g.stride_w - 1) // g.stride_w]
        cols = unfold(spread, (g.S, g.R), padding=(g.S - 1 - g.pad_h, g.R - 1 - g.pad_w))
        flt = wt.flip(2, 3).transpose(0, 1).reshape(g.C, -1)
        return flt, cols.transpose(0, 1).reshape(cols.shape[1], -1), lambda d: d.transpose(1, 0, 2, 3).reshape(g.C, -1)
    cols = unfold(xt, (g.S, g.R), padding=(g.pad_h, g.pad_w), stride=(g.stride_h, g.stride_w))
    return (dyt.reshape(g.N, g.K, -1).transpose(0, 1).reshape(g.K, -1), cols.transpose(1, 2).reshape(-1, cols.shape[1]),
            lambda d: d.reshape(g.K, -1))


def fma_chain(a, b):
    """The product as a chain of fused multiply-adds in fp32, term by term: what fp32 instructions do."""
    s = torch.zeros((a.shape[0], b.shape[1]), dtype=torch.float64)
    for r in range(a.shape[1]):
        s = (s + a[:, r, None] * b[r]).float().double()
    return s


def norm_error(got, ref):
    return float((got - ref).norm() / ref.norm())


SHORT = {
    "1x1 16->48": Geom(8, 16, 48, 64, 64, 1, 1),
    "1x1 64->32": Geom(8, 64, 32, 64, 64, 1, 1),
    "1x1 32->48": Geom(8, 32, 48, 64, 64, 1, 1),
    "1x1 16->80": Geom(4, 16, 80, 64, 64, 1, 1),
    "1x1 144->80": Geom(4, 144, 80, 64, 64, 1, 1),
    "3x3 16->32": Geom(2, 16, 32, 20, 14, 3, 3, 1, 1, 1, 1),
    "3x3 64->144": Geom(2, 64, 144, 14, 14, 3, 3, 1, 1, 1, 1),
    "3x3 256->256 split": Geom(1, 256, 256, 7, 7, 3, 3, 1, 1, 1, 1),
    "3x3 stride 2 32->16": Geom(4, 32, 16, 28, 28, 3, 3, 2, 2, 1, 1),
    "3x3 stride 2 16->80": Geom(4, 16, 80, 28, 28, 3, 3, 2, 2, 1, 1),
    # BWW over 16 to 196 pixels: every number of tiles around the limit of the short form, one and several partial sums
    "3x3 64->64 one tile": Geom(1, 64, 64, 4, 4, 3, 3, 1, 1, 1, 1),
    "3x3 512->256 one image": Geom(1, 512, 256, 7, 7, 3, 3, 1, 1, 1, 1),
    "3x3 64->80 @14": Geom(1, 64, 80, 14, 14, 3, 3, 1, 1, 1, 1),
    "3x3 80->64 two images": Geom(2, 80, 64, 8, 16, 3, 3, 1, 1, 1, 1),
    "3x3 stride 2 64->64 @14": Geom(1, 64, 64, 14, 14, 3, 3, 2, 2, 1, 1),
    "1x1 144->64 @7": Geom(1, 144, 64, 7, 7, 1, 1),
    "1x1 64->144 nine images": Geom(9, 64, 144, 14, 14, 1, 1),
}


@pytest.mark.parametrize("zeros", [0.0, 0.5, 0.8])
@pytest.mark.parametrize("name", SHORT)
def test_short_reductions_err_no_more_than_fp32_instructions(name, zeros):
    """Few non-zero products per output, where every rounding counts and no averaging over a long reduction helps: the error
    against 64 bits is no larger than that of a chain of fp32 multiply-adds over the same terms.  5 %: the products of pieces
    that are left out (root mean square 5e-9 of a product) beside one rounding of it (2.4e-8) are 3 % where an output has one
    product, and the two errors are those of 5000 outputs and more, 2 % of chance.  BWW with 4 % non-zero products has that few
    of them (16 pixels: none or one), so that the 3 % and what the products of one step cut off of each other (2^-24 of the largest,
    up to a rounding where two of them meet) are all there is beside the chain's own rounding: 10 %."""
    g = SHORT[name]
    x = stgen.relu_sparse(g.x_shape, zeros, 31) if zeros else stgen.normal(31, int(np.prod(g.x_shape))).reshape(g.x_shape).astype(np.float32)
    w = stgen.he_normal(g.w_shape, 32)
    dy = stgen.bernoulli_masked(g.y_shape, zeros, 33, 34)
    L = DeviceLayer(g, x, w, dy)
    for p in ("fwd", "bwi", "bww"):
        a, b, shape = as_products(g, x, w, dy, p)
        exact = a @ b
        got = torch.from_numpy(shape(getattr(L, p)(True)).astype(np.float64))
        err, chain = norm_error(got, exact), norm_error(fma_chain(a, b), exact)
        assert err <= (1.1 if p == "bww" else 1.05) * chain, f"{name} {p} {zeros}: {err:.3g}, fp32 instructions {chain:.3g}"


WIDE = {
    # kernels that take 32 reduced channels at a time, 3x3: 2, 3, 4 and 8 stages, split among workgroups and not, wavefronts without
    # channels of their own (80, 48), tiles of 64 and 128 pixels with ragged ends, tiles over many images, the larger halo, stride 2
    "64->80 33x31": Geom(8, 64, 80, 33, 31, 3, 3, 1, 1, 1, 1),
    "96->144 @14": Geom(24, 96, 144, 14, 14, 3, 3, 1, 1, 1, 1),
    "128->48 17x57": Geom(16, 128, 48, 17, 57, 3, 3, 1, 1, 1, 1),
    "64->64 3x5": Geom(2600, 64, 64, 3, 5, 3, 3, 1, 1, 1, 1),
    "128->64 31x57": Geom(16, 128, 64, 31, 57, 3, 3, 1, 1, 1, 1),
    "128->128 @56": Geom(6, 128, 128, 56, 56, 3, 3, 1, 1, 1, 1),
    "256->64 @28 pad 2": Geom(12, 256, 64, 28, 28, 3, 3, 1, 1, 2, 2),
    "stride 2 128->96 45x27": Geom(16, 128, 96, 45, 27, 3, 3, 2, 2, 1, 1),
    # 1x1 kernel: 1, 2, 3 and 8 stages of 64 channels, split and not, wavefronts without channels, ragged ends of the pixel numbering
    "1x1 64->256": Geom(4, 64, 256, 47, 45, 1, 1),
    "1x1 128->160": Geom(3, 128, 160, 41, 43, 1, 1),
    "1x1 192->144": Geom(4, 192, 144, 37, 29, 1, 1),
    "1x1 512->272 split": Geom(2, 512, 272, 39, 41, 1, 1),
    "1x1 160->48 ragged": Geom(5, 160, 48, 61, 57, 1, 1),
    "1x1 320->64 split": Geom(4, 320, 64, 67, 61, 1, 1),
    "1x1 1536->256 split, few workgroups": Geom(1, 1536, 256, 47, 45, 1, 1),
}


@pytest.mark.parametrize("value", [None, np.inf])
@pytest.mark.parametrize("name", WIDE)
def test_dense_forms_of_32_channels_at_a_time(name, value):
    """Values of very different size side by side, or a few infinities: each output within the bound of an fp32 sum."""
    g = WIDE[name]
    assert dense_kernel(desc_of(g)) == "32", "another kernel: test is void"
    x, w, dy = inputs(g, 37)
    if value is None:
        rng = np.random.default_rng(7)
        for t in (x, w, dy):
            t *= np.float32(2.0) ** rng.integers(-20, 21, t.shape).astype(np.float32)
    else:
        w[w == 0] = 0.25
        x[-1, -1, -1, -1] = x[0, 17, 1, 2] = dy[0, 0, 0, 0] = value
    check(g, x, w, dy, name)


@pytest.mark.parametrize("name", WIDE)
def test_outputs_stored_by_one_lane_and_replaced_by_another(name):
    """Finite results that the pieces cannot form (factors from 2^104 on): every output is stored, found non-finite by another lane of
    the wavefront and replaced.  The outputs hold ones before: a lane that looked too early would leave infinities behind."""
    g = WIDE[name]
    x, w, dy = inputs(g, 39)
    huge, small = np.float32(2.0 ** 110), np.float32(2.0 ** -60)
    for p, (a, b, c) in {"fwd": (x * huge, w * small, None), "bwi": (None, w * small, dy * huge), "bww": (x * huge, None, dy * small)}.items():
        ref, ref_abs = {"fwd": lambda: st_ref.conv_fwd(g, a, b), "bwi": lambda: st_ref.conv_bwi(g, c, b), "bww": lambda: st_ref.conv_bww(g, a, c)}[p]()
        L = DeviceLayer(g, a, b, c)
        L.fill = 1.0
        got = getattr(L, p)(True).astype(np.float64)
        assert np.isfinite(got).all(), f"{name} {p}"
        assert np.all(np.abs(got - ref) <= (terms(g)[p] + 3) * 2.0 ** -24 * ref_abs), f"{name} {p}"


@pytest.mark.parametrize("name", ["fwd", "bwi"])
def test_long_reductions_err_far_less_than_fp32_instructions(name):
    """2304 terms, reduced by one workgroup: a chain of fp32 multiply-adds rounds the running sum once per term, the dense form
    once per channel block of 144, and its twelve roundings per 16 terms are those of the block's sum, a quarter the size: (12 * 9 *
    16 / 16 + 16) against 2304 in variance, 0.23 in error.  0.28 leaves a fifth for what products of pieces cut off of each other;
    with the large products on the running sum (two roundings per 16 terms) it is 0.35."""
    g = Geom(32, 256, 16, 56, 56, 3, 3, 1, 1, 1, 1) if name == "fwd" else Geom(32, 16, 256, 56, 56, 3, 3, 1, 1, 1, 1)
    w = stgen.he_normal(g.w_shape, 61)
    shape = g.x_shape if name == "fwd" else g.y_shape
    t = stgen.normal(62, int(np.prod(shape))).reshape(shape).astype(np.float32)
    L = DeviceLayer(g, t if name == "fwd" else None, w, t if name == "bwi" else None)
    one = Geom(1, g.C, g.K, 56, 56, 3, 3, 1, 1, 1, 1)               # the first image
    a, b, flat = as_products(one, t[:1], w, t[:1], name)
    exact = a @ b
    got = torch.from_numpy(flat(getattr(L, name)(True)[:1]).astype(np.float64))
    err, chain = norm_error(got, exact), norm_error(fma_chain(a, b), exact)
    assert err <= 0.28 * chain, f"{err:.3g}, fp32 instructions {chain:.3g}"


def microseconds(fn):
    """Best of five bursts of ten calls."""
    best = float("inf")
    for _ in range(5):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(10):
            fn()
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) * 100)
    return best


@pytest.mark.parametrize("name", ["fwd", "bwi", "bww"])
@pytest.mark.parametrize("g", [Geom(4, 128, 128, 56, 56, 3, 3, 1, 1, 1, 1), Geom(4, 128, 128, 56, 56, 3, 3, 2, 2, 1, 1),
                               Geom(8, 256, 256, 56, 56, 1, 1)], ids=["3x3", "stride 2", "1x1"])
def test_time_of_values_at_the_ends_of_the_range(g, name):
    """Vanishing values, one (a decayed filter weight, the gradient of a sample the network is sure of) or all of them, cost
    nothing.  Values from 2^104 on, infinities and NaN make the wavefronts they reach compute their tiles a second time on slower
    instructions: a few times the usual time and no more, whatever the number of such values."""
    import paper_1911_10175_amd as st
    from tests.gpu_harness import desc_of, workspace

    gen = torch.Generator(device="cuda").manual_seed(3)
    t = {"x": torch.randn((g.N, g.C // 16, g.H, g.W, 16), device="cuda", generator=gen),
         "w": torch.randn((g.K // 16, g.C // 16, g.S, g.R, 16, 16), device="cuda", generator=gen),
         "dy": torch.randn((g.N, g.K // 16, g.OH, g.OW, 16), device="cuda", generator=gen)}
    a, b, out = {"fwd": ("x", "w", "dy"), "bwi": ("dy", "w", "x"), "bww": ("x", "dy", "w")}[name]
    d, o = desc_of(g), torch.empty_like(t[out])
    ws = workspace(d, {"fwd": st.ST_PASS_FWD, "bwi": st.ST_PASS_BWI, "bww": st.ST_PASS_BWW}[name], True)
    entry = getattr(st, f"st_conv_{name}_dense")

    def time_with(which, value, everywhere):
        ops = {k: t[k].clone() for k in (a, b)}
        if everywhere:
            ops[which].fill_(value)
        elif value is not None:
            ops[which].view(-1)[ops[which].numel() // 3] = value
        return microseconds(lambda: entry(d, ops[a], ops[b], o, ws))

    time_with(a, None, False)
    usual = time_with(a, None, False)
    # 1.5: two measurements of the same work.  10: the usual time, then 16/6 of its matrix time at fp32 rate without the overlap
    # of staging and arithmetic that makes the usual time; measured 1.4 to 7 (before such tiles were computed by
    # wavefronts, lane by lane: one value 10 to 150)
    for which in (a, b):
        for value, everywhere, factor in ((1e-35, False, 1.5), (1e-42, False, 1.5), (1e-35, True, 1.5), (float("inf"), False, 10), (float("inf"), True, 10),
                                          (1e36, False, 10), (float("nan"), False, 10)):
            us = time_with(which, value, everywhere)
            assert us <= factor * usual + 5, f"{name} {value} in {which}{' everywhere' if everywhere else ''}: {us:.0f} us, usually {usual:.0f}"


@pytest.mark.parametrize("g", [Geom(3, 16, 64, 61, 53, 1, 1), Geom(3, 16, 80, 61, 53, 1, 1), Geom(5, 48, 32, 57, 61, 1, 1), Geom(5, 64, 32, 57, 61, 1, 1),
                               Geom(2, 80, 16, 203, 151, 1, 1), Geom(2, 32, 48, 203, 151, 1, 1)], ids=lambda g: f"{g.C}to{g.K} {g.H}x{g.W}")
def test_1x1_layers_of_few_produced_channels(g):
    """Either side of the lines between the two 1x1 kernels, FWD and, with the roles of the channels exchanged, BWI;
    ragged ends of the pixel numbering."""
    x = stgen.relu_sparse(g.x_shape, 0.5, 51)
    w = stgen.he_normal(g.w_shape, 52)
    flip = Geom(g.N, g.K, g.C, g.H, g.W, 1, 1)          # its BWI is the same product
    L, M = DeviceLayer(g, x, w, None), DeviceLayer(flip, None, w.transpose(1, 0, 2, 3), x)
    ref = np.einsum("kc,nchw->nkhw", w[:, :, 0, 0].astype(np.float64), x.astype(np.float64))
    mag = np.einsum("kc,nchw->nkhw", np.abs(w[:, :, 0, 0]).astype(np.float64), np.abs(x).astype(np.float64))
    for got in (L.fwd(True), M.bwi(True)):
        assert np.all(np.abs(got - ref) <= (g.C + 3) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("g", [Geom(2, 64, 144, 30, 26, 3, 3, 1, 1, 1, 1), Geom(1, 320, 320, 20, 22, 3, 3, 1, 1, 1, 1), Geom(3, 48, 160, 17, 19, 3, 3, 2, 2, 1, 1),
                               Geom(2, 16, 352, 41, 37, 1, 1), Geom(2, 336, 272, 9, 11, 1, 1)], ids=lambda g: f"{g.R}x{g.S}/{g.stride_w} {g.C}to{g.K}")
def test_bww_with_numbers_of_filter_groups_that_do_not_divide_the_chip(g):
    """3, 25, 3, 3 and 9 groups of filters: partial gradients over unequal shares of the tiles."""
    x, w, dy = inputs(g, 23)
    L = DeviceLayer(g, x, w, dy)
    ref, ref_abs = st_ref.conv_bww(g, x, dy)
    bound = (g.N * g.OH * g.OW + 3) * 2.0 ** -24 * ref_abs
    for form in (True, "auto"):
        assert np.all(np.abs(L.bww(form) - ref) <= bound), form


@pytest.mark.parametrize("g,form", [(Geom(4, 208, 256, 9, 9, 3, 3, 1, 1, 1, 1), False), (Geom(1, 256, 256, 28, 28, 3, 3, 1, 1, 1, 1), False), (Geom(2, 336, 192, 12, 12, 3, 3, 1, 1, 1, 1), False),
                                    (Geom(3, 80, 48, 37, 53, 3, 3, 1, 1, 1, 1), True),
                                    (Geom(4, 64, 128, 14, 14, 3, 3, 1, 1, 1, 1), True), (Geom(2, 64, 64, 56, 56, 3, 3, 1, 1, 1, 1), True),
                                    (Geom(8, 512, 512, 14, 14, 3, 3, 1, 1, 1, 1), True)], ids=lambda v: f"{v.C}to{v.K} {v.H}" if isinstance(v, Geom) else "")
def test_bww_auto_takes_the_faster_form_of_launches_bound_by_partial_gradients(g, form):
    """Half zeros: bit for bit the zero-skipping form (x tested) where every one of at most 128 workgroups has one tile and
    the partial gradients are 24 MB and more, the dense form elsewhere."""
    x, w, dy = inputs(g, 29)
    L = DeviceLayer(g, x, None, dy)
    got = L.bww("auto", raw=True)
    assert torch.equal(got, L.bww(form, raw=True))
    assert not torch.equal(got, L.bww(not form, raw=True)), "forms indistinguishable: test is void"


@pytest.mark.parametrize("g,form", [(Geom(8, 64, 64, 56, 56, 3, 3, 2, 2, 1, 1), "dy"), (Geom(15, 96, 160, 33, 41, 3, 3, 2, 2, 1, 1), "dy"),
                                    (Geom(16, 96, 160, 33, 41, 3, 3, 2, 2, 1, 1), True), (Geom(32, 64, 64, 56, 56, 3, 3, 2, 2, 1, 1), True),
                                    (Geom(32, 32, 64, 74, 74, 3, 3, 2, 2, 1, 1), "dy"), (Geom(32, 64, 48, 60, 60, 3, 3, 2, 2, 1, 1), "dy"),
                                    (Geom(32, 80, 80, 48, 48, 3, 3, 2, 2, 1, 1), "dy")], ids=lambda v: f"{v.N}x{v.C}to{v.K}" if isinstance(v, Geom) else "")
def test_bww_auto_of_stride_2_layers(g, form):
    """Bit for bit the dense form from 750 million multiply-adds on (740 and 790 million here) with 64 and more channels that fill at
    least half of whole groups, else the dy-testing one."""
    x, w, dy = inputs(g, 43)
    L = DeviceLayer(g, x, None, dy)
    got = L.bww("auto", raw=True)
    assert torch.equal(got, L.bww(form, raw=True))
    assert not torch.equal(got, L.bww("dy" if form is True else True, raw=True)), "forms indistinguishable: test is void"


def test_images_taken_one_by_one_are_read_with_the_filter_copy_of_the_whole_call():
    """So many channels that a launch takes one image (its sample offsets are kept in int): by itself, with 8 tiles, an image would be
    left to the kernel of 16 channels at a time, the two of the call are not.  1024 channels hold values, few enough for a reference."""
    N, C, K, H, W = 2, 260096, 64, 9, 113
    d = st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(51)
    x = torch.zeros((N, C // 16, H, W, 16), device="cuda")
    blocks = torch.arange(5, C // 16, C // 16 // 64, device="cuda")[:64]
    x[:, blocks] = torch.randn((N, 64, H, W, 16), device="cuda", generator=g)
    w = torch.randn((K // 16, C // 16, 3, 3, 16, 16), device="cuda", generator=g)
    ws = torch.empty((st.st_conv_workspace_bytes(d, st.ST_PASS_FWD, True) + 3) // 4, device="cuda")
    y = torch.full((N, K // 16, H, W, 16), float("nan"), device="cuda")
    st.st_conv_fwd_dense(d, x, w, y, ws)
    torch.cuda.synchronize()
    xr = x[:, blocks].double().permute(1, 4, 0, 2, 3).reshape(1024, N, H, W)                    # [c][n][h][w]
    xr = torch.nn.functional.pad(xr, (1, 1, 1, 1))
    wr = w[:, blocks].double().permute(2, 3, 0, 5, 1, 4).reshape(3, 3, K, 1024)
    ref = sum(wr[v, u] @ xr[:, :, v:v + H, u:u + W].reshape(1024, -1) for v in range(3) for u in range(3))
    mag = sum(wr[v, u].abs() @ xr[:, :, v:v + H, u:u + W].abs().reshape(1024, -1) for v in range(3) for u in range(3))
    got = y.double().permute(1, 4, 0, 2, 3).reshape(K, -1)
    assert bool(((got - ref).abs() <= (9 * 1024 + 3) * 2.0 ** -24 * mag).all())


@pytest.mark.parametrize("zeros", [(0.5, 0.0), (0.5, 0.5), (0.5, 0.7), (0.5, 0.9), (0.9, 0.9)])
def test_error_of_bww_auto_of_stride_2_layers(zeros):
    """The dense form's error against 64 bits beside that of testing dy, which multiplies and adds with one rounding of the sum.  A product
    of pieces is rounded by itself before it joins the sum: 2.4e-8 of it (2^-24 / sqrt(3), averaged over the mantissas), as much of the
    norm for terms of independent signs.  Up to 70 % zeros the rounding of longer sums is the larger part and the dense form errs less."""
    g = Geom(16, 96, 160, 33, 41, 3, 3, 2, 2, 1, 1)
    x = stgen.relu_sparse(g.x_shape, zeros[0], 61)
    dy = stgen.bernoulli_masked(g.y_shape, zeros[1], 62, 63)
    L = DeviceLayer(g, x, None, dy)
    ref = st_ref.conv_bww(g, x, dy)[0]
    err = {f: np.linalg.norm(L.bww(f) - ref) / np.linalg.norm(ref) for f in ("auto", "dy")}
    print(f"stride 2 BWW, zeros {zeros}: {err}")
    assert err["auto"] <= 1.1 * np.hypot(err["dy"], 2.4e-8), err
    if zeros[1] <= 0.7:
        assert err["auto"] <= err["dy"], err


@pytest.mark.parametrize("g", [Geom(1, 16, 32, 3, 32100, 3, 3, 1, 1, 1, 1), Geom(1, 32, 16, 32100, 2, 3, 3, 1, 1, 1, 1), Geom(2, 80, 48, 2, 31999, 3, 3, 1, 1, 1, 1)],
                         ids=lambda g: f"{g.H}x{g.W}")
def test_bww_of_images_with_long_sides(g):
    """Either side of the line from which rows and columns are no longer compared as packed pairs of 16 bits."""
    x, w, dy = inputs(g, 47)
    ref, ref_abs = st_ref.conv_bww(g, x, dy)
    off = np.abs(DeviceLayer(g, x, None, dy).bww(True) - ref)
    assert np.all(off <= (g.N * g.OH * g.OW + 3) * 2.0 ** -24 * ref_abs)


@pytest.mark.parametrize("g,px,pdy,form", [(Geom(4, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.85, 0.5, True), (Geom(4, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.5, 0.85, True),
                                           (Geom(4, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.85, 0.85, False), (Geom(4, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.0, 0.98, "dy"),
                                           (Geom(4, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.94, 0.0, True), (Geom(3, 64, 128, 24, 24, 3, 3, 1, 1, 1, 1), 0.85, 0.5, False)],
                         ids=lambda v: f"N={v.N}" if isinstance(v, Geom) else str(v))
def test_bww_auto_above_75_percent_zeros(g, px, pdy, form):
    """From 128 million multiply-adds on (N = 4) bit for bit the dense form up to 96 % zeros in the sparser operand where at least 5 % of the products are
    not zero; in smaller launches, or with fewer products, the zero-skipping form that tests it."""
    x = stgen.relu_sparse(g.x_shape, px, 71) if px else stgen.normal(71, int(np.prod(g.x_shape))).reshape(g.x_shape).astype(np.float32)
    dy = stgen.bernoulli_masked(g.y_shape, pdy, 72, 73)
    L = DeviceLayer(g, x, None, dy)
    got = L.bww("auto", raw=True)
    assert torch.equal(got, L.bww(form, raw=True))
    assert not torch.equal(got, L.bww(False if form is True else True, raw=True)), "forms indistinguishable: test is void"


@pytest.mark.parametrize("zeros", [0.0, 0.7])
@pytest.mark.parametrize("g", [Geom(2, 256, 256, 28, 28, 3, 3, 1, 1, 1, 1), Geom(1, 512, 512, 14, 14, 3, 3, 1, 1, 1, 1), Geom(5, 144, 304, 8, 12, 3, 3, 1, 1, 1, 1),
                               Geom(3, 80, 48, 37, 53, 3, 3, 1, 1, 1, 1), Geom(16, 128, 128, 28, 28, 3, 3, 1, 1, 1, 1), Geom(4, 432, 48, 19, 19, 3, 3, 1, 1, 2, 2), Geom(3, 48, 32, 17, 181, 3, 3, 1, 1, 1, 1)],
                         ids=lambda g: f"{g.N}x{g.C}to{g.K} {g.H}" if isinstance(g, Geom) else "")
def test_bww_of_two_teams_in_a_workgroup(g, zeros):
    """Workgroups of 1, 2, 4 and 5 tiles, of one team or (3x80->48, 3x48->32 with an odd number of teams: the last one has no partner) two, channel counts
    that leave wavefronts without any; the direct call and the self-selecting one, whose final sum is another launch; an infinity in the last tiles."""
    x = stgen.relu_sparse(g.x_shape, zeros, 81) if zeros else stgen.normal(81, int(np.prod(g.x_shape))).reshape(g.x_shape).astype(np.float32)
    dy = stgen.bernoulli_masked(g.y_shape, 0.5, 82, 83)
    L = DeviceLayer(g, x, None, dy)
    ref, ref_abs = st_ref.conv_bww(g, x, dy)
    bound = (g.N * g.OH * g.OW + 3) * 2.0 ** -24 * ref_abs
    first = L.bww(True)
    assert np.all(np.abs(first - ref) <= bound)
    assert np.all(np.abs(L.bww("auto") - ref) <= bound)
    assert np.array_equal(first, L.bww(True)), "two runs differ"
    x[-1, 3, -2, 1] = np.inf
    ref = st_ref.conv_bww(g, x, dy)[0]
    got = DeviceLayer(g, x, None, dy).bww(True)
    fine = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fine) and np.all(np.abs(got[fine] - ref[fine]) <= bound[fine])


@pytest.mark.parametrize("g,err", [(Geom(2, 256, 256, 28, 28, 3, 3, 1, 1, 1, 1), 5.07e-8), (Geom(1, 512, 512, 14, 14, 3, 3, 1, 1, 1, 1), 3.81e-8),
                                   (Geom(5, 144, 304, 8, 12, 3, 3, 1, 1, 1, 1), 4.24e-8), (Geom(27, 32, 256, 14, 8, 3, 3, 1, 1, 1, 1), 4.27e-8),
                                   (Geom(16, 128, 128, 28, 28, 3, 3, 1, 1, 1, 1), 6.03e-8), (Geom(3, 80, 48, 37, 53, 3, 3, 1, 1, 1, 1), 5.53e-8),
                                   (Geom(3, 48, 32, 17, 181, 3, 3, 1, 1, 1, 1), 5.41e-8)], ids=lambda v: f"{v.N}x{v.C}to{v.K} {v.H}" if isinstance(v, Geom) else "")
def test_error_of_bww_of_few_tiles(g, err):
    """No more than with a partial gradient for every four wavefronts, which is what the limits were measured with (these inputs; the sums have a fixed
    order).  Sums of two teams that are rounded before the final sum add up to half of that again."""
    x, dy = stgen.relu_sparse(g.x_shape, 0.5, 81), stgen.bernoulli_masked(g.y_shape, 0.5, 82, 83)
    ref = st_ref.conv_bww(g, x, dy)[0]
    off = np.linalg.norm(DeviceLayer(g, x, None, dy).bww(True) - ref) / np.linalg.norm(ref)
    assert off <= 1.03 * err, off
