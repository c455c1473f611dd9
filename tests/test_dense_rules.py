"""Choices of the dense forms that their workspace queries tell (host side only)."""
import pytest

import paper_1911_10175_amd as st
from tests.kernel_choice import bww_line, dense_kernel, f16_pieces


def partials(N, C, K, H, W, stride=1):
    d = st.ConvDesc(N, C, K, H, W, 3, 3, stride, stride, 1, 1)
    need = st.st_conv_workspace_bytes(d, st.ST_PASS_BWW, True)
    assert need % (K * C * 9 * 4) == 0
    return need // (K * C * 9 * 4)


def test_no_more_partial_gradients_than_the_longest_workgroup_calls_for():
    # 784 tiles of 4 x 8 pixels: at most 512 workgroups would take two each, and 392 do
    assert partials(8, 64, 64, 56, 56) == 392
    assert partials(32, 64, 64, 56, 56) == 448                  # 3136 tiles, seven each
    assert partials(32, 256, 256, 56, 56) == 32                 # 16 workgroups for the filters alone
    # fewer tiles than workgroups: one each
    assert partials(2, 64, 64, 28, 28) == 56
    assert partials(2, 112, 48, 8, 214, 2) == 56


def test_few_tiles_of_many_filters_go_straight_to_the_gradient():
    assert partials(1, 512, 512, 7, 7) == 0
    assert partials(1, 512, 512, 14, 14) == 7                   # seven tiles
    assert partials(1, 64, 64, 7, 7) == 2                       # the chip would be empty


@pytest.mark.parametrize("C,K", [(16, 352), (64, 144), (320, 320), (448, 512), (176, 368), (1536, 1792), (80, 1280)])
def test_no_more_workgroups_than_fit_on_the_chip(C, K):
    """256 compute units hold two workgroups of the 3x3 kernel each, or one of the 1x1 kernel; one workgroup more would run by itself."""
    groups = -(-C // 64) * -(-K // 64)
    assert 1 <= partials(32, C, K, 28, 28) * groups <= 512 or groups > 256
    cw, kw = (128 if n > 64 else 64 for n in (C, K))
    groups = -(-C // cw) * -(-K // kw)
    d = st.ConvDesc(32, C, K, 28, 28, 1, 1)
    need = st.st_conv_workspace_bytes(d, st.ST_PASS_BWW, True)
    assert need % (K * C * 4) == 0 and max(1, need // (K * C * 4)) * groups <= 256


def bytes_per_filter_element(N, C, K, H, W):
    """4: the copy of the 1x1 kernel on fp32 instructions, 6: three bf16 pieces (K is padded to whole groups of 128)."""
    d = st.ConvDesc(N, C, K, H, W, 1, 1)
    return st.st_conv_workspace_bytes(d, st.ST_PASS_FWD, True) / ((K + 127) // 128 * 128 * C)


def test_1x1_layers_of_few_produced_channels_stay_on_fp32_instructions():
    assert [bytes_per_filter_element(16, 16, k, 112, 112) for k in (16, 32, 48, 64, 80)] == [4, 4, 4, 4, 6]
    assert [bytes_per_filter_element(16, 32, k, 112, 112) for k in (16, 32, 48)] == [4, 4, 6]
    assert [bytes_per_filter_element(32, c, 32, 80, 80) for c in (48, 64, 80, 256)] == [4, 6, 4, 4]
    assert [bytes_per_filter_element(4, c, 256, 56, 56) for c in (16, 256)] == [6, 6]
    assert bytes_per_filter_element(1, 256, 256, 14, 14) == 4          # few pixels


def test_1x1_layers_of_64_to_127_workgroups_leave_fp32_instructions_from_1536_channels_on():
    def fp32(*layer):
        return bytes_per_filter_element(*layer) == 4               # (else pieces, and partial outputs)
    assert [fp32(32, c, 512, 7, 7) for c in (1024, 1472, 1536, 2048)] == [True, True, False, False]      # 100 workgroups
    assert [fp32(n, 2048, 512, 7, 7) for n in (19, 21)] == [True, False]                                 # 60, 68
    assert [fp32(18, 2048, k, 28, 28) for k in (48, 64)] == [True, True]                                 # 111, at most 64 produced


def test_the_switching_points_of_the_self_selecting_entry_points_can_be_asked_for():
    F, B = st.ST_PASS_FWD_AUTO, st.ST_PASS_BWI_AUTO
    ask = st.st_conv_sparse_threshold
    vgg = st.ConvDesc(16, 256, 256, 56, 56, 3, 3, 1, 1, 1, 1)
    assert ask(vgg, F) == 950 and ask(vgg, B) == 950
    # one main kernel with fewer than 128 reduced channels (FWD: C, BWI: K); two kernels
    mixed = st.ConvDesc(16, 64, 128, 56, 56, 3, 3, 1, 1, 1, 1)
    assert ask(mixed, F) == 650 and ask(mixed, B) == 850
    # never: stride 2, 1x1; always: geometries without a tiled dense form
    assert ask(st.ConvDesc(8, 128, 128, 56, 56, 3, 3, 2, 2, 1, 1), F) == 1001
    assert ask(st.ConvDesc(8, 64, 256, 56, 56, 1, 1), B) == 1001
    assert ask(st.ConvDesc(1, 16, 16, 9, 9, 5, 5, 1, 1, 2, 2), F) == 0
    assert ask(st.ConvDesc(0, 16, 16, 9, 9, 3, 3), F) == -1 and ask(vgg, st.ST_PASS_BWW_AUTO) == -1
    # never below what the form itself needs to beat fp32 instructions
    for d in (vgg, mixed):
        for auto, direct in ((F, st.ST_PASS_FWD), (B, st.ST_PASS_BWI)):
            assert ask(d, auto) >= ask(d, direct)


def kernel_names(d, direct, auto):
    names = []
    for p in (direct, auto):
        try:
            names.append(st.st_conv_kernel_name(d, p))
        except st.StConvError:
            names.append("")
    return names


def test_layers_without_a_filter_copy_have_no_kernel_that_reads_one():
    """The one-launch kernels of small layers read the layer's own filters and no copy is written for them; the kernel that holds both
    forms reads the copy.  No layer may have both."""
    seen = {"direct": 0, "both forms": 0}
    for N in (1, 8, 32, 256, 516):
        for C in (32, 48, 64, 128, 240):
            for K in (128, 256, 512):
                for H, W in ((1, 1), (2, 2), (2, 4), (5, 3), (7, 5), (7, 7), (14, 14), (60, 1), (100, 1), (1, 100), (56, 56)):
                    for pad in (0, 1, 2):
                        if min(H, W) + 2 * pad < 3:
                            continue
                        fwd = st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, pad, pad)
                        bwi = st.ConvDesc(N, K, C, fwd.OH, fwd.OW, 3, 3, 1, 1, 2 - pad, 2 - pad)
                        for d, passes in ((fwd, (st.ST_PASS_FWD, st.ST_PASS_FWD_AUTO)), (bwi, (st.ST_PASS_BWI, st.ST_PASS_BWI_AUTO))):
                            direct, auto = kernel_names(d, *passes)
                            assert not (direct.startswith("fwd_direct") and auto), (d, direct, auto)
                            seen["direct"] += direct.startswith("fwd_direct")
                            seen["both forms"] += auto != ""
    assert min(seen.values()) > 100


def test_switching_points_of_small_layers_are_those_of_larger_ones():
    F = st.ST_PASS_FWD_AUTO
    assert st.st_conv_sparse_threshold(st.ConvDesc(32, 48, 512, 7, 5, 3, 3), F) == 650
    assert st.st_conv_sparse_threshold(st.ConvDesc(516, 128, 128, 1, 1, 3, 3, 1, 1, 1, 1), F) == 950
    assert st.st_conv_sparse_threshold(st.ConvDesc(1, 64, 64, 16, 16, 3, 3, 1, 1, 1, 1), F) == 850


@pytest.mark.parametrize("N,C,K,H,W,one_launch", [
    # whole runs of four pixels: up to 120 million multiply-adds, 96 with one channel block into more than four
    (1, 64, 64, 56, 56, True), (1, 64, 64, 57, 60, False), (1, 32, 512, 28, 28, True), (1, 16, 512, 36, 36, True), (1, 16, 128, 80, 80, False),
    (1, 16, 64, 112, 112, True),
    # rows that are no multiple of four pixels, down to single pixels
    (1, 512, 512, 7, 7, True), (95, 64, 64, 5, 5, True), (124, 64, 64, 5, 5, False), (25, 64, 64, 32, 1, True), (50, 64, 64, 32, 1, False),
    (135, 16, 48, 32, 1, True), (271, 16, 48, 32, 1, False), (101, 128, 128, 1, 1, True), (203, 128, 128, 1, 1, False), (6, 256, 256, 16, 2, False)])
def test_one_launch_kernels_of_small_layers(N, C, K, H, W, one_launch):
    """Where the zero-skipping form is one launch: a run of pixels costs the same whether the row has them or not."""
    d = st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)
    assert st.st_conv_kernel_name(d, st.ST_PASS_FWD).startswith("fwd_direct_kernel") == one_launch


def shares(N, C, K, H, W):
    """Of a dense FWD launch of less than eight channel blocks: the copy, then the partial outputs of all but the first."""
    copy = (K + 127) // 128 * 128 * C * 9 * 6
    need = st.st_conv_workspace_bytes(st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1), st.ST_PASS_FWD, True)
    return 1 + (need - (copy + 255) // 256 * 256) // (N * K * H * W * 4) if need > copy else 1


def test_single_blocks_are_shared_out_where_their_partial_outputs_are_small():
    assert shares(3, 80, 48, 37, 53) == 5 and shares(2, 112, 48, 40, 40) == 7          # 1.1 and 0.6 MB each
    assert shares(50, 64, 64, 7, 7) == 4                                              # 0.6 MB
    assert shares(25, 80, 128, 16, 16) == 2 and shares(7, 48, 64, 37, 37) == 1           # 3.3 MB; three blocks


@pytest.mark.parametrize("N,C,K,H,W,kernel", [
    # two stages: two shares that fit the chip as two workgroups a compute unit, and a few that do not; whole where there are enough
    (5, 64, 128, 56, 56, "32"), (10, 64, 64, 56, 56, "16"), (180, 64, 192, 7, 7, "16"), (32, 64, 64, 56, 56, "32"),
    # launches that the kernel of 16 channels leaves whole: up to four stages, more
    (200, 64, 128, 9, 9, "16"), (25, 64, 256, 8, 44, "16"), (83, 128, 256, 9, 9, "16"), (50, 128, 192, 13, 13, "32"), (80, 256, 256, 9, 9, "32"),
    (488, 256, 64, 9, 7, "16"), (1152, 512, 64, 5, 5, "32"),
    # the longest of many shares, with 64 produced channels and with more
    (39, 512, 64, 14, 14, "16"), (9, 512, 128, 28, 28, "32"),
    # two shares of tiles of 128 pixels that are cut short by their halo
    (627, 256, 64, 7, 7, "16"), (77, 256, 48, 20, 20, "16"), (692, 256, 64, 7, 7, "32"), (372, 128, 48, 14, 7, "32"), (90, 320, 128, 14, 14, "32"), (93, 192, 64, 17, 17, "32")])
def test_split_launches_take_the_faster_dense_kernel(N, C, K, H, W, kernel):
    assert dense_kernel(st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)) == kernel
    assert dense_kernel(st.ConvDesc(N, K, C, H, W, 3, 3, 1, 1, 1, 1), bwi=True) == kernel


@pytest.mark.parametrize("N,C,K,H,W,kernel", [
    # at most 64 produced channels: up to two workgroups a compute unit, not in what three of the other kernel hold; short reductions never
    (329, 160, 48, 14, 14, "32"), (339, 160, 48, 14, 14, "16"), (496, 1024, 64, 14, 14, "16"), (522, 1024, 64, 14, 14, "32"), (32, 128, 48, 56, 56, "16"),
    # outputs beyond the last-level cache, few reduced channels
    (8, 192, 640, 112, 112, "32"), (8, 192, 768, 112, 112, "16"), (8, 512, 1024, 112, 112, "32"), (64, 192, 128, 112, 112, "32"),
    (32, 64, 256, 112, 112, "32"), (32, 64, 64, 56, 56, "lds"), (32, 32, 32, 80, 80, "fp32")])
def test_1x1_launches_take_the_faster_dense_kernel(N, C, K, H, W, kernel):
    assert dense_kernel(st.ConvDesc(N, C, K, H, W, 1, 1)) == kernel
    assert dense_kernel(st.ConvDesc(N, K, C, H, W, 1, 1), bwi=True) == kernel


def test_1x1_shares_of_launches_near_a_workgroup_per_compute_unit():
    def count(N, C, K):
        copy = (K + 127) // 128 * 128 * C * 6
        need = st.st_conv_workspace_bytes(st.ConvDesc(N, C, K, 14, 14, 1, 1), st.ST_PASS_FWD, True)
        return 1 if need == copy else 1 + (need - copy) // (N * K * 14 * 14 * 4)
    # 250 workgroups, 262, 287, 400
    assert [count(n, 512, 48) for n in (163, 171, 187, 261)] == [2, 1, 1, 1]
    assert [count(n, 1024, 48) for n in (163, 171, 187, 261)] == [2, 3, 3, 1]
    assert [count(n, 512, 256) for n in (41, 42, 46)] == [2, 1, 1] and [count(n, 2048, 256) for n in (41, 42, 46)] == [2, 3, 3]


@pytest.mark.parametrize("N,C,K,H,W,half", [
    # seven blocks and more, whole launches or shares of more than three stages; short reductions, short shares and few workgroups stay
    (20, 112, 256, 76, 76, True), (17, 304, 128, 35, 35, True), (11, 400, 96, 17, 31, True), (21, 112, 128, 29, 29, True), (32, 80, 128, 56, 56, False),
    (11, 272, 96, 17, 31, False), (9, 112, 128, 68, 23, False), (1, 112, 128, 28, 28, False), (20, 112, 32, 76, 76, True), (5, 112, 32, 76, 76, False)])
def test_odd_numbers_of_channel_blocks_on_f16_pieces(N, C, K, H, W, half):
    d = st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)
    assert (dense_kernel(d), f16_pieces(d)) == (("32", True) if half else ("16", False))
    if half:
        assert st.st_conv_sparse_threshold(d, st.ST_PASS_FWD_AUTO) == 950


@pytest.mark.parametrize("N,C,K,H,W,stride,pad,bwi,size", [
    # an odd number of reduced channel blocks, whole and in shares, at stride 2; at most 32 produced channels
    (6, 464, 688, 7, 21, 1, 1, False, 24097536), (6, 464, 688, 7, 21, 1, 1, True, 25569792), (2, 592, 720, 20, 20, 1, 1, True, 30566400),
    (7, 560, 592, 128, 4, 1, 0, False, 19353600), (6, 400, 96, 76, 76, 2, 1, False, 6091776), (92, 288, 400, 9, 3, 1, 1, True, 8294400),
    (10, 512, 32, 84, 84, 1, 1, False, 3538944), (18, 592, 32, 3, 233, 1, 1, False, 10533888), (7, 224, 16, 49, 199, 1, 2, False, 1548288),
    (13, 32, 704, 239, 23, 1, 1, True, 4866048), (3, 16, 336, 223, 54, 1, 0, True, 4634496), (77, 736, 32, 5, 63, 1, 0, False, 12301824)])
def test_workspaces_that_sufficed_suffice(N, C, K, H, W, stride, pad, bwi, size):
    """Sizes that the query has told for these layers with the kernel of 16 channels at a time: a program may have kept them, and the kernel of
    32 channels, with shares of its own, must not ask for more."""
    d = st.ConvDesc(N, C, K, H, W, 3, 3, stride, stride, pad, pad)
    assert st.st_conv_workspace_bytes(d, st.ST_PASS_BWI if bwi else st.ST_PASS_FWD, True) <= size


@pytest.mark.parametrize("N,C,K,H,W,kernel", [(4, 112, 32, 174, 174, "16"), (4, 144, 32, 174, 174, "16"), (4, 256, 32, 174, 174, "32"), (5, 112, 32, 174, 174, "32"),
                                              (41, 112, 32, 56, 56, "32"), (42, 112, 32, 56, 56, "32")])
def test_tiles_of_256_pixels_that_take_one_round_more(N, C, K, H, W, kernel):
    """479 workgroups of the kernel of 16 channels are one round of the chip, 525 of the other, whose tiles strips of 174 columns cut short, two."""
    assert dense_kernel(st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)) == kernel
    assert dense_kernel(st.ConvDesc(N, K, C, H, W, 3, 3, 1, 1, 1, 1), bwi=True) == kernel


@pytest.mark.parametrize("N,C,K,H,W,line", [
    # one to three tiles of the zero-skipping form a partial gradient, nine to 119 of these; four tiles, eight gradients, 120 and more, one dense tile a gradient; small launches
    (2, 256, 256, 28, 28, 750), (6, 128, 128, 28, 28, 750), (12, 128, 256, 28, 28, 750), (16, 512, 256, 7, 7, 750), (8, 256, 256, 28, 28, 960),
    (4, 512, 512, 14, 14, 960), (4, 128, 128, 40, 40, 960), (4, 64, 128, 24, 24, 960), (16, 256, 256, 56, 56, 960), (2, 64, 128, 24, 24, 750), (1, 256, 256, 28, 28, 250)])
def test_switching_point_of_the_self_selecting_bww(N, C, K, H, W, line):
    assert bww_line(st.ConvDesc(N, C, K, H, W, 3, 3, 1, 1, 1, 1)) == line
