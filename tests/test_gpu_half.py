"""Dense kernels that form fp32 products from two f16 pieces (long reductions): the error of an ordinary layer, and values of the sizes
where the pieces' five exponent bits end.  Every test here needs an MI355X."""
import numpy as np
import pytest
import torch

import stgen
from oracle import st_ref
from oracle.st_ref import Geom

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1911_10175_amd as st
    from tests.gpu_harness import DeviceLayer, desc_of, workspace
    from tests.kernel_choice import bww_f16_pieces, f16_pieces
    from tests.test_gpu_split import as_products, check, fma_chain, inputs, norm_error

# whole launches of 4 and 5 stages, two shares, tiles of 64 and 128 pixels (the larger halo too), tiles over many images, stride 2
GEOMS = {
    "128->128 @56": Geom(6, 128, 128, 56, 56, 3, 3, 1, 1, 1, 1),
    "160->80 33x31": Geom(18, 160, 80, 33, 31, 3, 3, 1, 1, 1, 1),
    "256->144 @14": Geom(44, 256, 144, 14, 14, 3, 3, 1, 1, 1, 1),
    "128->64 @57x61": Geom(11, 128, 64, 57, 61, 3, 3, 1, 1, 1, 1),
    "192->48 3x5": Geom(2600, 192, 48, 3, 5, 3, 3, 1, 1, 1, 1),
    # at most 32 produced channels, tiles of 256 pixels: rows that fit and not, tiny images, an odd last block
    "128->32 @57x61": Geom(24, 128, 32, 57, 61, 3, 3, 1, 1, 1, 1),
    "144->16 3x5": Geom(4600, 144, 16, 3, 5, 3, 3, 1, 1, 1, 1),
    "16->112 @28, BWI": Geom(100, 16, 112, 28, 28, 3, 3, 1, 1, 1, 1),
    # an odd last block of 16 channels: 112 whole, 400 in shares, stride 2
    "112->144 @28": Geom(22, 112, 144, 28, 28, 3, 3, 1, 1, 1, 1),
    "400->96 17x31, shares": Geom(11, 400, 96, 17, 31, 3, 3, 1, 1, 1, 1),
    "176->48 @40 pad 2": Geom(22, 176, 48, 40, 40, 3, 3, 1, 1, 2, 2),
    "stride 2 144->112 45x27": Geom(64, 144, 112, 45, 27, 3, 3, 2, 2, 1, 1),
    "stride 2 160->160 45x27": Geom(32, 160, 160, 45, 27, 3, 3, 2, 2, 1, 1),
}


def half_passes(g):
    d = desc_of(g)
    return [p for p, bwi in (("fwd", False), ("bwi", True)) if f16_pieces(d, bwi)]


def corr(g, x, w, dy, p):
    return st_ref.conv_fwd(g, x, w) if p == "fwd" else st_ref.conv_bwi(g, dy, w)


def within_fp32_sum(g, x, w, dy, label):
    L = DeviceLayer(g, x, w, dy)
    passes = half_passes(g)
    assert passes, "another kernel: test is void"
    for p in passes:
        ref, mag = corr(g, x, w, dy, p)
        n = (g.C if p == "fwd" else g.K) * g.R * g.S
        off, bound = np.abs(getattr(L, p)(True).astype(np.float64) - ref), (n + 3) * 2.0 ** -24 * mag + n * 2.0 ** -150
        assert np.all(off <= bound), f"{label} {p}: {np.max(off / np.maximum(bound, 1e-300))} of the bound"


@pytest.mark.parametrize("small", [2.0 ** -13, 2.0 ** -27, 2.0 ** -33, 2.0 ** -60, 2.0 ** -120])
@pytest.mark.parametrize("name", GEOMS)
def test_images_and_filters_of_very_different_scale(name, small):
    """Every other image (its outputs share tiles with those of its neighbours), then every other filter, then every other reduced channel is
    smaller by a factor on either side of what the pieces hold beside the larger ones.  Each output within the bound of an fp32 sum: those
    that only small values take part in are as exact as the others."""
    g = GEOMS[name]
    x, w, dy = inputs(g, 71)
    s = np.float32(small)
    scaled = x.copy(), dy.copy()
    for t in scaled:
        t[1::2] *= s
    within_fp32_sum(g, scaled[0], w, scaled[1], f"{name} images {small}")
    w2 = w.copy()
    w2[1::2, ::2] *= s
    w2[::2, 1::2] *= s
    xs, dys = x.copy(), dy.copy()
    xs[:, 1::2] = 0                                     # even rows: the large filters only; odd rows: the small ones only
    dys[:, 1::2] = 0
    within_fp32_sum(g, xs, w2, dys, f"{name} filters {small}")
    xs[:, 1::2] = x[:, 1::2] * s                        # and with factors that make up for it
    dys[:, 1::2] = dy[:, 1::2] * s
    within_fp32_sum(g, xs, w2 / s if small > 2.0 ** -100 else w2, dys, f"{name} both {small}")


@pytest.mark.parametrize("name", ["128->128 @56", "stride 2 160->160 45x27"])
def test_zeros_and_tensors_of_extreme_scale(name):
    g = GEOMS[name]
    x, w, dy = inputs(g, 73)
    within_fp32_sum(g, 0 * x, w, 0 * dy, "zeros")
    within_fp32_sum(g, x, 0 * w, dy, "zero filters")
    one = np.zeros_like(x), np.zeros_like(dy)
    for t in one:
        t[-1, 5, 1, 1] = 2.0 ** -126                    # nothing else: hardly any sample sees it
    within_fp32_sum(g, one[0], w, one[1], "one value")
    for a, b in ((2.0 ** 100, 2.0 ** -90), (2.0 ** -110, 2.0 ** 90), (2.0 ** -128, 2.0 ** 110)):
        within_fp32_sum(g, x * np.float32(a), w * np.float32(b), dy * np.float32(a), f"{a} {b}")


@pytest.mark.parametrize("name", GEOMS)
def test_values_far_above_the_sampled_ones(name):
    """A few values that no sample is likely to see, 2^4 to 2^60 times the others: h is infinite from 2^5 on and such outputs are computed
    again."""
    g = GEOMS[name]
    for big in (2.0 ** 4, 2.0 ** 9, 2.0 ** 60):
        x, w, dy = inputs(g, 75)
        for t in (x, dy):
            t.reshape(-1)[[7, t.size // 2, t.size - 3]] = np.float32(5 * big)
        within_fp32_sum(g, x, w, dy, f"{name} {big}")
        x, w, dy = inputs(g, 75)
        w[0, 0, 0, 0] = w[-1, -1, -1, -1] = np.float32(big)
        within_fp32_sum(g, x, w, dy, f"{name} filter {big}")


@pytest.mark.parametrize("above", [2 ** 6, 2 ** 10, 2 ** 14, 2 ** 15, 2 ** 16])
@pytest.mark.parametrize("name", ["256->144 @14", "128->64 @57x61"])
def test_a_second_pass_for_values_above_the_sampled_ones(name, above):
    """A few values above what the first scale holds: the second one holds them up to 2^15 times the sampled ones, beyond them outputs are
    computed with fp32 multiply-adds, and an infinity among them leaves the others as they are."""
    g = GEOMS[name]
    x, w, dy = inputs(g, 111)
    for t in (x, dy):
        t.reshape(-1)[5::40009] = 3 * above
    within_fp32_sum(g, x, w, dy, f"{name} {above}")
    y = DeviceLayer(g, x, w, dy).fwd(True)
    x.reshape(-1)[x.size // 2] = np.inf
    with_inf = DeviceLayer(g, x, w, dy).fwd(True)
    fine = np.isfinite(with_inf)
    assert 0 < np.count_nonzero(~fine) <= 9 * g.K and np.abs(with_inf - y)[fine].max() <= 1e-6 * np.abs(y).max()


@pytest.mark.parametrize("p", ["fwd", "bwi"])
def test_time_of_a_few_values_above_the_sampled_ones(p):
    """One in 10^6 had taken four to six times as long, as a launch waits for the one tile that is computed with fp32 multiply-adds.  Twice the time is
    what multiplying a workgroup all over costs; half of that again for noise."""
    gen = torch.Generator(device="cuda").manual_seed(103)
    d = st.ConvDesc(32, 128, 128, 28, 28, 3, 3, 1, 1, 1, 1)
    assert f16_pieces(d, p == "bwi")
    w = torch.randn((8, 8, 3, 3, 16, 16), device="cuda", generator=gen)
    a, out = torch.randn((32, 8, 28, 28, 16), device="cuda", generator=gen), torch.empty((32, 8, 28, 28, 16), device="cuda")
    fn, ws = (st.st_conv_fwd_dense, workspace(d, st.ST_PASS_FWD, True)) if p == "fwd" else (st.st_conv_bwi_dense, workspace(d, st.ST_PASS_BWI, True))

    def time(a):
        took = []
        for _ in range(20):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            fn(d, a, w, out, ws)
            end.record()
            torch.cuda.synchronize()
            took.append(start.elapsed_time(end))
        return sorted(took)[5]

    usual = time(a)
    a *= torch.where(torch.rand(a.shape, device="cuda", generator=gen) < 1e-6, 1000.0, 1.0)
    took = time(a)
    assert took <= 3 * usual, (took, usual)


def time_of_fwd(d, x, w, y):
    ws, took = workspace(d, st.ST_PASS_FWD, True), []
    for _ in range(20):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        st.st_conv_fwd_dense(d, x, w, y, ws)
        end.record()
        torch.cuda.synchronize()
        took.append(start.elapsed_time(end))
    return sorted(took)[5]


@pytest.mark.parametrize("name", ["128->128 @56", "128->64 @57x61", "144->16 3x5", "16->112 @28, BWI", "400->96 17x31, shares", "stride 2 160->160 45x27"])
def test_channels_without_filters(name):
    """Produced channels that padding has left without filters, and values below the pieces' range that make small outputs suspect: zeros, but where an
    infinity meets a filter of zero; a channel with one filter, however small, is as exact as the others."""
    g = GEOMS[name]
    x, w, dy = inputs(g, 115)
    dead = np.arange(g.K) % 16 >= 4
    if half_passes(g)[0] == "fwd":
        w[dead] = 0
        w[5, 0, 0, 0] = np.float32(2.0 ** -70)
    else:
        w[:, np.arange(g.C) % 16 >= 4] = 0
        w[0, 5, 0, 0] = np.float32(2.0 ** -70)
    for t in (x, dy):
        t.reshape(-1)[::997] = np.float32(2.0 ** -60)
    within_fp32_sum(g, x, w, dy, name)
    x[0, 0, 1, 1] = dy[0, 0, 1, 1] = np.inf
    L = DeviceLayer(g, x, w, dy)
    for p in half_passes(g):
        with np.errstate(invalid="ignore"):
            ref = corr(g, x, w, dy, p)[0]
        got = getattr(L, p)(True)
        assert np.array_equal(np.isnan(got[0]), np.isnan(ref[0])), f"{name} {p}"


@pytest.mark.parametrize("every", [1, 101, 9973])
@pytest.mark.parametrize("name", ["128->128 @56", "192->48 3x5", "256->144 @14", "112->144 @28", "400->96 17x31, shares", "176->48 @40 pad 2"])
def test_a_few_outputs_that_small_values_may_matter_to(name, every):
    """Values of all sizes down to 2^-40, all or some of them: the outputs near zero are computed one by one, where there are more than eight of 32 x 32 with
    fp32 multiply-adds."""
    g = GEOMS[name]
    x, w, dy = inputs(g, 119)
    rng = np.random.default_rng(121)
    for t in (x, dy):
        some = t.reshape(-1)[::every]
        some *= np.exp2(-40 * rng.random(some.size)).astype(np.float32)
    within_fp32_sum(g, x, w, dy, f"{name} {every}")


@pytest.mark.parametrize("name", ["128->128 @56", "128->64 @57x61", "192->48 3x5", "256->144 @14", "400->96 17x31, shares", "176->48 @40 pad 2"])
def test_pixels_that_meet_no_value(name):
    """Rows of an image without values, and values below the pieces' range, or above it, in others: zeros, but where an infinite filter meets them; a pixel that
    meets one value, however small, is as exact as the others."""
    g = GEOMS[name]
    for above in (1.0, 3.0 * 2 ** 10):
        x, w, dy = inputs(g, 117)
        for t in (x, dy):
            t.reshape(-1)[::997] = np.float32(2.0 ** -60)
            t.reshape(-1)[11::40009] *= np.float32(above)
            t[1::2, :, : t.shape[2] - 2] = 0
            t[0, :, t.shape[2] // 2:] = 0
            t[0, 1, -1, -1] = np.float32(2.0 ** -70)
        within_fp32_sum(g, x, w, dy, f"{name} {above}")
    w[3, 5, 1, 1] = np.inf
    L = DeviceLayer(g, x, w, dy)
    for p in half_passes(g):
        with np.errstate(invalid="ignore"):
            ref = corr(g, x, w, dy, p)[0]
        assert np.array_equal(np.isnan(getattr(L, p)(True)), np.isnan(ref)), f"{name} {p}"


@pytest.mark.parametrize("N,C,K,H", [(16, 128, 64, 112), (32, 128, 128, 28)])
def test_time_of_pixels_that_meet_no_value(N, C, K, H):
    """As below, three to six times the time.  Looking for these takes each workgroup a second look at its input."""
    gen = torch.Generator(device="cuda").manual_seed(107)
    d = st.ConvDesc(N, C, K, H, H, 3, 3, 1, 1, 1, 1)
    assert f16_pieces(d)
    w = torch.randn((K // 16, C // 16, 3, 3, 16, 16), device="cuda", generator=gen)
    x, y = torch.randn((N, C // 16, H, H, 16), device="cuda", generator=gen), torch.empty((N, K // 16, H, H, 16), device="cuda")
    usual = time_of_fwd(d, x, w, y)
    x[:, :, : H // 2] = 0
    x.view(-1)[::10007] *= 2.0 ** -60
    took = time_of_fwd(d, x, w, y)
    assert took <= 2 * usual, (took, usual)


@pytest.mark.parametrize("N,C,K,H", [(32, 256, 32, 56), (16, 128, 64, 112), (32, 128, 128, 28)])
def test_time_of_channels_without_filters(N, C, K, H):
    """A value below the pieces' range in the same tile had all of these computed again with fp32 multiply-adds: two to five times the time."""
    gen = torch.Generator(device="cuda").manual_seed(105)
    d = st.ConvDesc(N, C, K, H, H, 3, 3, 1, 1, 1, 1)
    assert f16_pieces(d)
    w = torch.randn((K // 16, C // 16, 3, 3, 16, 16), device="cuda", generator=gen)
    x, y = torch.randn((N, C // 16, H, H, 16), device="cuda", generator=gen), torch.empty((N, K // 16, H, H, 16), device="cuda")
    usual = time_of_fwd(d, x, w, y)
    w[-1, ..., 4:] = 0
    x.view(-1)[::10007] = 2.0 ** -60
    took = time_of_fwd(d, x, w, y)
    assert took <= 1.5 * usual, (took, usual)


def test_infinities_and_nan():
    for name in ("128->64 @57x61", "256->144 @14"):
        g = GEOMS[name]
        for value in (np.inf, np.nan):
            x, w, dy = inputs(g, 77)
            w[w == 0] = 0.25
            x[-1, 3, 2, 2] = dy[0, 1, 0, 1] = value
            check(g, x, w, dy, f"{name} {value}")


@pytest.mark.parametrize("zeros", [0.0, 0.5, 0.9])
@pytest.mark.parametrize("channels", [128, 256])
def test_error_of_ordinary_layers(channels, zeros):
    """Beside a chain of fp32 multiply-adds, which rounds the running sum once per non-zero term.  In units of half a squared rounding of
    the whole sum: three taps' 12 roundings (a group of 8 products each) of a sum that is 1/T of the whole, T of them, and T joins, T = 9 C /
    96, so 12 + T against 9 C (1 - zeros); what the pieces leave out adds 7.5e-8, three roundings of a product (2.4e-8).  A fifth more for what
    products cut off of each other."""
    N = {128: 6, 256: 6}[channels]
    g, one = Geom(N, channels, 128, 56, 56, 3, 3, 1, 1, 1, 1), Geom(1, channels, 128, 56, 56, 3, 3, 1, 1, 1, 1)
    assert f16_pieces(desc_of(g)), "another kernel: test is void"
    w = stgen.he_normal(g.w_shape, 82)
    x = stgen.relu_sparse(g.x_shape, zeros, 81) if zeros else stgen.normal(81, int(np.prod(g.x_shape))).reshape(g.x_shape).astype(np.float32)
    L = DeviceLayer(g, x, w, None)
    a, b, flat = as_products(one, x[:1], w, x[:1], "fwd")
    rows = slice(0, 16)                                 # a block of produced channels
    exact = (a @ b)[rows]
    got = torch.from_numpy(flat(L.fwd(True)[:1]).astype(np.float64))[rows]
    err, chain = norm_error(got, exact), norm_error(fma_chain(a[rows], b), exact)
    T = 9 * channels / 96
    bound = 1.2 * np.hypot(np.sqrt((12 + T) / (9 * channels * (1 - zeros))) * chain, 7.5e-8)
    assert err <= bound, f"{err:.3g}, bound {bound:.3g}, fp32 instructions {chain:.3g}"


# BWW: (N, C, K, H, W, pad), 48 and more tiles for a workgroup.  Even and odd numbers of tiles, 4 x 8 and 2 x 14 pixels, ragged ends, channels that
# fill no whole group of 64, shares of unequal length
BWW = {
    "1024->1024 @56x55, 49 tiles": (1, 1024, 1024, 56, 55, 1),
    "1040->528 @14, 56": (24, 1040, 528, 14, 14, 1),
    "528->1040 37x41 pad 2": (3, 528, 1040, 37, 41, 2),
    "768->784 @31x29 pad 0": (5, 768, 784, 31, 29, 0),
}


def bww_inputs(N, C, K, H, W, pad, seed):
    d = st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, pad, pad)
    assert bww_f16_pieces(d), "another kernel: test is void"
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.relu(torch.randn((N, C // 16, H, W, 16), device="cuda", generator=gen))
    dy = torch.randn((N, K // 16, d.OH, d.OW, 16), device="cuda", generator=gen)
    dy *= torch.rand(dy.shape, device="cuda", generator=gen) >= 0.5
    return d, x, dy


def bww_result(d, x, dy):
    dw = torch.full((d.K // 16, d.C // 16, 3, 3, 16, 16), float("nan"), device="cuda")
    st.st_conv_bww_dense(d, x, dy, dw, workspace(d, st.ST_PASS_BWW, True))
    torch.cuda.synchronize()
    return dw.permute(2, 3, 0, 5, 1, 4).reshape(3, 3, d.K, d.C).double()


def bww_exact(d, x, dy):
    """Result and sum of magnitudes in 64 bits, [v][u][k][c]."""
    def plain(t):
        return t.double().permute(1, 4, 0, 2, 3).reshape(t.shape[1] * 16, t.shape[0], t.shape[2], t.shape[3])
    xp = torch.nn.functional.pad(plain(x), (d.pad_w, d.pad_w, d.pad_h, d.pad_h))
    dyf = plain(dy).reshape(d.K, -1)
    ref, mag = (torch.empty((3, 3, d.K, d.C), dtype=torch.float64, device="cuda") for _ in range(2))
    for v in range(3):
        for u in range(3):
            cols = xp[:, :, v:v + d.OH, u:u + d.OW].reshape(d.C, -1).t()
            ref[v, u], mag[v, u] = dyf @ cols, dyf.abs() @ cols.abs()
    return ref, mag


def bww_within_fp32_sum(d, x, dy, label):
    got, (ref, mag) = bww_result(d, x, dy), bww_exact(d, x, dy)
    n = d.N * d.OH * d.OW
    off, bound = (got - ref).abs(), (n + 3) * 2.0 ** -24 * mag + n * 2.0 ** -150
    assert bool((off <= bound).all()), f"{label}: {float((off / bound.clamp_min(1e-300)).max())} of the bound"


@pytest.mark.parametrize("small", [1.0, 2.0 ** -13, 2.0 ** -27, 2.0 ** -60, 2.0 ** -120])
@pytest.mark.parametrize("name", BWW)
def test_bww_channels_and_pixels_of_very_different_scale(name, small):
    """Every other channel of x and of dy, or of the first halves of the blocks, then every other row of pixels: gradients that only small
    values take part in are as exact as the others."""
    d, x, dy = bww_inputs(*BWW[name], 91)
    xs, dys = x.clone(), dy.clone()
    xs[..., 1::2] *= small
    dys[..., ::2] *= small
    bww_within_fp32_sum(d, xs, dy, f"{name} x {small}")
    bww_within_fp32_sum(d, x, dys, f"{name} dy {small}")
    if small > 2.0 ** -100:
        bww_within_fp32_sum(d, xs, dys / small, f"{name} both {small}")
    xs, dys = x.clone(), dy.clone()
    xs[:, :, 1::2] *= small
    dys[:, :, 1::2] = 0
    bww_within_fp32_sum(d, xs, dys, f"{name} rows {small}")


@pytest.mark.parametrize("name", ["1024->1024 @56x55, 49 tiles", "1040->528 @14, 56"])
def test_bww_values_outside_the_pieces_and_zeros(name):
    d, x, dy = bww_inputs(*BWW[name], 93)
    bww_within_fp32_sum(d, torch.zeros_like(x), dy, "zeros")
    for a, b in ((2.0 ** 100, 2.0 ** -90), (2.0 ** -110, 2.0 ** 90)):
        bww_within_fp32_sum(d, x * a, dy * b, f"{a} {b}")
    for big in (2.0 ** 4, 2.0 ** 9, 2.0 ** 60):                 # no sample is likely to see them; h is infinite from 2^5 on
        xb = x.clone()
        xb.view(-1)[[7, x.numel() // 2, x.numel() - 3]] = 5 * big
        bww_within_fp32_sum(d, xb, dy, f"{big}")
    one = torch.zeros_like(x)
    one.view(-1)[x.numel() // 3] = 2.0 ** -126
    bww_within_fp32_sum(d, one, dy, "one value")
    xi = x.clone()
    xi.view(-1)[x.numel() // 2] = float("inf")
    got, ref = bww_result(d, xi, dy), bww_exact(d, xi, dy)[0]
    assert torch.equal(torch.isfinite(got), torch.isfinite(ref))
    fine = torch.isfinite(ref)
    assert bool(((got - ref)[fine].abs() <= 1e-6 * ref[fine].abs().max()).all())


def test_bww_workgroups_that_sample_few_products_stay_on_bf16_pieces():
    """95 % zeros in x and in dy: the error that bf16 pieces leave, which two f16 pieces could not reach."""
    d, x, dy = bww_inputs(1, 1024, 1024, 56, 55, 1, 95)
    gen = torch.Generator(device="cuda").manual_seed(96)
    x *= torch.rand(x.shape, device="cuda", generator=gen) < 0.1
    dy *= torch.rand(dy.shape, device="cuda", generator=gen) < 0.1
    ref = bww_exact(d, x, dy)[0]
    err = float((bww_result(d, x, dy) - ref).norm() / ref.norm())
    # 8 terms a gradient: 2.4e-8 for each rounding of a product or a sum, of which a join is one every fourth tile; f16 pieces alone leave out 7.5e-8
    assert err <= 7e-8, err


def test_bww_of_one_product_in_18_stays_on_bf16_pieces():
    """Half zeros in x, 89 % in dy, and values whose pieces leave 2^-22 of every product out, whatever the signs: 2.4e-7 of the norm."""
    d, x, dy = bww_inputs(1, 1024, 1024, 56, 55, 1, 99)
    gen = torch.Generator(device="cuda").manual_seed(100)
    v = 1 + 2.0 ** -11 - 2.0 ** -22
    x = (x > 0) * v
    dy = torch.sign(dy) * (torch.rand(dy.shape, device="cuda", generator=gen) < 0.22) * v
    ref = bww_exact(d, x, dy)[0]
    err = float((bww_result(d, x, dy) - ref).norm() / ref.norm())
    # 170 terms a gradient, a rounding of 2.4e-8 to 3.5e-8 each eight of them and each join
    assert err <= 1.7e-7, err


@pytest.mark.parametrize("N,C,K", [(2, 256, 256), (6, 128, 128), (8, 128, 256)])
def test_self_selecting_bww_with_few_products_a_partial_gradient(N, C, K):
    """77 % zeros in both: no further off than the zero-skipping form, whose sums are exact but for some roundings there (dense 4 to 6 % more)."""
    d = st.ConvDesc(N, C, K, 28, 28, 3, 3, 1, 1, 1, 1)
    gen = torch.Generator(device="cuda").manual_seed(101)
    x = torch.relu(torch.randn((N, C // 16, 28, 28, 16), device="cuda", generator=gen) - 0.739)
    dy = torch.randn((N, K // 16, 28, 28, 16), device="cuda", generator=gen)
    dy *= torch.rand(dy.shape, device="cuda", generator=gen) >= 0.77
    ref = bww_exact(d, x, dy)[0]

    def err(fn, ps):
        dw = torch.full((K // 16, C // 16, 3, 3, 16, 16), float("nan"), device="cuda")
        fn(d, x, dy, dw, workspace(d, ps, False))
        torch.cuda.synchronize()
        return float((dw.permute(2, 3, 0, 5, 1, 4).reshape(3, 3, K, C).double() - ref).norm() / ref.norm())

    assert err(st.st_conv_bww_auto, st.ST_PASS_BWW_AUTO) <= 1.005 * err(st.st_conv_bww, st.ST_PASS_BWW)


@pytest.mark.parametrize("name", ["1024->1024 @56x55, 49 tiles", "528->1040 37x41 pad 2"])
def test_bww_of_channels_without_values(name):
    """Channels that padding or ReLU has left without values, and values below the pieces' range in the other operand: the zeros are exact, other
    gradients as exact as ever, and an infinity meets the zeros as it would in a plain sum (NaN)."""
    d, x, dy = bww_inputs(*BWW[name], 97)
    dead = torch.arange(16, device="cuda") >= 3
    for a, b in ((x, dy), (dy, x)):
        a, b = a.clone(), b.clone()
        a[..., dead] = 0
        b.view(-1)[::4099] = 2.0 ** -60
        xs, dys = (a, b) if a.shape == x.shape and b.shape == dy.shape else (b, a)
        bww_within_fp32_sum(d, xs, dys, name)
    a = dy.clone()
    a[..., dead] = 0
    x[-1, 0, 1, 1, 2] = float("inf")
    got, ref = bww_result(d, x, a), bww_exact(d, x, a)[0]
    assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isfinite(got), torch.isfinite(ref))


@pytest.mark.parametrize("name", BWW)
@pytest.mark.parametrize("share,few", [(1e-3, 4), (0.3, 64)])
def test_bww_gradients_below_what_lost_values_may_matter_to(name, share, few):
    """A part of the values of some channels is below the pieces' range, so that now and then a gradient is too, few of a wavefront's (computed one by
    one) or, with these channels' other values made small as well, all of them (the workgroup starts again)."""
    d, x, dy = bww_inputs(*BWW[name], 99)
    gen = torch.Generator(device="cuda").manual_seed(100)
    small = torch.rand(x.shape, device="cuda", generator=gen) < share
    small[..., few:] = False
    x = torch.where(small, x * 2.0 ** -40, x)
    bww_within_fp32_sum(d, x, dy, name)
    x[:, 1, ..., :4] *= 2.0 ** -18
    bww_within_fp32_sum(d, x, dy, name)


@pytest.mark.parametrize("case", ["channels without values", "heavy tails", "one outlier in 10^6"])
def test_time_of_bww_on_values_that_are_not_normal(case):
    """Each of these had taken four to eight times as long, as one workgroup that computes its gradients again with fp32 multiply-adds is all it
    takes.  Twice the time is what starting again on bf16 pieces costs; half of that again for noise."""
    gen = torch.Generator(device="cuda").manual_seed(101)
    d = st.ConvDesc(16, 64, 64, 224, 224, 3, 3, 1, 1, 1, 1)
    assert bww_f16_pieces(d)
    dw, ws = torch.empty((4, 4, 3, 3, 16, 16), device="cuda"), workspace(d, st.ST_PASS_BWW, True)

    def time(x, dy):
        took = []
        for _ in range(12):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            st.st_conv_bww_dense(d, x, dy, dw, ws)
            end.record()
            torch.cuda.synchronize()
            took.append(start.elapsed_time(end))
        return sorted(took)[3]

    x = torch.randn((16, 4, 224, 224, 16), device="cuda", generator=gen)
    dy = torch.randn((16, 4, 224, 224, 16), device="cuda", generator=gen)
    usual = time(x, dy)
    if case == "channels without values":
        x[..., 10:] = 0
        dy.view(-1)[::1000003] = 2.0 ** -60
    elif case == "heavy tails":
        for t in (x, dy):
            t /= torch.sqrt(-torch.log(torch.rand(t.shape, device="cuda", generator=gen).clamp_min(1e-30)))
    else:
        x *= torch.where(torch.rand(x.shape, device="cuda", generator=gen) < 1e-6, 100.0, 1.0)
    assert time(x, dy) <= 3 * usual


ROUNDING = 2.4e-8                                   # of one rounding to 24 bits, in the root mean square, and what two pieces leave out of a product
PIECES = 7.5e-8


def stages_of(d, bwi):
    """Reduced channels of the longest share of a launch, from its workspace: the filter copy (a multiple of 256 bytes), then the partial outputs."""
    Ci, Ko, px = (d.K, d.C, d.H * d.W) if bwi else (d.C, d.K, d.OH * d.OW)
    need = st.st_conv_workspace_bytes(d, st.ST_PASS_BWI if bwi else st.ST_PASS_FWD, True)
    extra = max(0, need - (Ko + 127) // 128 * 128 * Ci * 9 * 6)
    shares = 1 + extra // (4 * d.N * Ko * px)
    return -(-(-(-Ci // 32)) // shares) * 32


@pytest.mark.parametrize("name", GEOMS)
def test_error_of_every_kernel_on_ordinary_values(name):
    """Every column-block width, halo size, stride and kind of last stage.  Terms of independent signs: the three taps of 32 channels of a sum round 12 times on the
    way up (6.5 roundings of the whole), T = C / 32 * 3 sums join one after the other ((T + 1) / 2), and the pieces leave out theirs.  A quarter more
    for what products cut off of each other.  Without one of the cross products it would be 3e-4."""
    g = GEOMS[name]
    x, w, dy = inputs(g, 87)
    L = DeviceLayer(g, x, w, dy)
    passes = half_passes(g)
    assert passes, "another kernel: test is void"
    for p in passes:
        ref = corr(g, x, w, dy, p)[0]
        T = stages_of(desc_of(g), p == "bwi") // 32 * 3
        bound = 1.25 * np.hypot(np.sqrt(6.5 + (T + 1) / 2) * ROUNDING, PIECES)
        err = np.linalg.norm(getattr(L, p)(True) - ref) / np.linalg.norm(ref)
        assert err <= bound, f"{p}: {err:.3g}, bound {bound:.3g}"


@pytest.mark.parametrize("name", BWW)
def test_error_of_bww_on_ordinary_values(name):
    """Both tile shapes.  A pair of tiles rounds 8 times on the way up (4.5), T / 2 pairs join."""
    d, x, dy = bww_inputs(*BWW[name], 103)
    splits = max(1, st.st_conv_workspace_bytes(d, st.ST_PASS_BWW, True) // (d.K * d.C * 36))
    tiles = d.N * min(-(-d.OH // h) * -(-d.OW // w) for h, w in ((4, 8), (2, 14)))
    pairs = -(-(-(-tiles // splits)) // 2)
    got, ref = bww_result(d, x, dy), bww_exact(d, x, dy)[0]
    bound = 1.25 * np.hypot(np.sqrt(4.5 + (pairs + 1) / 2) * ROUNDING, PIECES)
    err = float((got - ref).norm() / ref.norm())
    assert err <= bound, f"{err:.3g}, bound {bound:.3g}"
