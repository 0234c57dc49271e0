"""GPU parity of the direct CONV's tile shapes and fetch paths against the
oracle (same bar as test_parity_conv: max|dY| / RMS(Y_ref) <= 2e-2, the bf16
rounding of the output): edges of the 64- and 128-pixel tiles and of the 48-,
64-, 80-, 128- and 160-filter ones, one to many slices of 64 columns, runs of
channels that are and are not whole slices, more taps than the in-image bit
mask holds, padding wider than the kernel, several conv groups, several tiles
per workgroup, and columns split over workgroups."""
import pytest

import paper_1807_11091_amd as sa
from test_parity_conv import conv_case

pytestmark = pytest.mark.gpu

D = {"path": {sa.CONV_DIRECT}}


def T(pixels, filters, slices, one_tap):
    """k_conv_tile (four fetching wavefronts) in this shape, `slices` in LDS."""
    return {"path": {sa.CONV_DIRECT}, "ksplit": 1, "direct_tile": (pixels, filters, 4, slices, one_tap)}


CASES = [
    # N, Cin, H, W, A, C, D, stride, pad, groups, kind, keep
    ((1, 64, 1, 1, 1, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # one output, one slice
    ((1, 128, 9, 7, 65, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # 63 pixels, 65 filters, two slices
    ((1, 192, 13, 5, 63, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # 65 pixels, three slices
    ((3, 64, 9, 9, 33, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # a slice per tap
    ((3, 64, 8, 10, 17, 3, 3, 1, 3, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # padding wider than the kernel
    ((2, 64, 5, 1, 20, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # one pixel wide
    ((2, 128, 15, 13, 70, 3, 3, 2, 1, 2, sa.FILTER, 0.7), T(64, 64, 4, 1)),  # two groups of 64 channels, stride 2
    ((1, 64, 1, 1, 40, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(64, 64, 4, 0)),  # image smaller than the kernel
    ((1, 64, 2, 1, 40, 5, 5, 1, 2, 1, sa.FILTER, 1.0), D),
    ((1, 128, 1, 3, 40, 3, 3, 1, 2, 2, sa.FILTER, 1.0), T(64, 64, 4, 1)),
    ((2, 64, 11, 12, 40, 5, 5, 2, 2, 1, sa.FILTER, 1.0), D),  # 25 taps, stride 2
    ((2, 8, 15, 16, 24, 7, 7, 1, 3, 1, sa.FILTER, 1.0), T(64, 64, 4, 0)),  # 49 taps of 8 channels
    ((30, 64, 9, 9, 90, 7, 5, 1, 2, 1, sa.FILTER, 1.0), T(64, 64, 4, 0)),  # 35 taps of 64 channels
    ((2, 72, 9, 11, 51, 3, 3, 1, 1, 3, sa.FILTER, 0.7), T(64, 64, 4, 0)),  # runs of 24 channels, three groups
    ((2, 96, 9, 11, 50, 3, 3, 2, 1, 1, sa.FILTER, 0.7), T(64, 64, 4, 0)),  # runs of 96: slices across taps
    ((20, 64, 28, 28, 154, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(64, 160, 3, 1)),  # 154 filters
    ((40, 64, 31, 29, 130, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 160, 2, 1)),  # many tiles of one slice
    ((30, 64, 56, 56, 38, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # 38 filters, one slice
    ((48, 64, 28, 29, 77, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(128, 80, 2, 1)),  # 77 filters
    ((24, 128, 28, 28, 128, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(128, 128, 3, 1)),
    ((9, 64, 20, 21, 200, 1, 1, 2, 0, 1, sa.FILTER, 1.0), T(64, 64, 4, 1)),  # 1x1 of stride 2
    ((16, 256, 56, 56, 20, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(128, 48, 2, 1)),  # 20 filters, four slices
    ((20, 64, 32, 32, 77, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 128, 2, 1)),  # 77 filters, one slice
    ((32, 24, 56, 56, 77, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(128, 80, 2, 0)),  # runs of 24 and 72 channels over the same shapes
    ((16, 24, 28, 28, 154, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 160, 3, 0)),
    ((15, 72, 32, 32, 300, 1, 1, 1, 0, 1, sa.FILTER, 1.0), T(64, 160, 2, 0)),
    ((25, 72, 28, 28, 100, 3, 3, 1, 1, 1, sa.FILTER, 1.0), T(128, 128, 3, 0)),
    # every shape over several conv groups, mostly with more tiles than the GPU
    # holds workgroups (a workgroup's range then runs on from group to group),
    # for slices within one tap and across taps; at least 40 columns, for the
    # reason given at FOOTPRINT (8 columns: 13 times the RMS, 0.026 by rounding alone)
    ((38, 576, 17, 17, 24, 1, 1, 1, 0, 3, sa.FILTER, 1.0), T(64, 64, 4, 1)),
    ((22, 216, 32, 31, 60, 1, 1, 1, 0, 3, sa.FILTER, 1.0), T(64, 64, 4, 0)),
    ((57, 256, 28, 29, 76, 1, 1, 1, 0, 2, sa.FILTER, 1.0), T(128, 48, 2, 1)),
    ((78, 200, 32, 32, 8, 3, 3, 1, 0, 1, sa.FILTER, 1.0), T(128, 48, 2, 0)),
    ((147, 400, 17, 17, 16, 3, 3, 1, 0, 2, sa.FILTER, 1.0), T(128, 48, 2, 0)),
    ((39, 256, 32, 33, 130, 1, 1, 1, 0, 2, sa.FILTER, 1.0), T(128, 80, 2, 1)),
    ((53, 120, 40, 41, 195, 1, 1, 2, 0, 3, sa.FILTER, 1.0), T(128, 80, 2, 0)),
    ((49, 192, 32, 32, 390, 3, 3, 2, 0, 3, sa.FILTER, 1.0), T(64, 160, 3, 1)),
    ((9, 120, 20, 20, 390, 1, 1, 1, 0, 3, sa.FILTER, 1.0), T(64, 160, 3, 0)),
    ((21, 128, 56, 55, 260, 1, 1, 2, 0, 2, sa.FILTER, 1.0), T(64, 160, 2, 1)),
    ((22, 80, 31, 32, 260, 1, 1, 1, 0, 2, sa.FILTER, 1.0), T(64, 160, 2, 0)),
    ((55, 192, 20, 20, 288, 3, 3, 2, 1, 3, sa.FILTER, 1.0), T(128, 128, 3, 1)),
    ((98, 320, 32, 32, 176, 3, 3, 2, 1, 2, sa.FILTER, 1.0), T(128, 128, 3, 0)),
    ((10, 128, 40, 41, 192, 1, 1, 1, 0, 2, sa.FILTER, 1.0), T(64, 128, 2, 1)),
    ((22, 144, 31, 32, 195, 1, 1, 1, 0, 3, sa.FILTER, 1.0), T(64, 128, 2, 0)),
    ((4, 512, 7, 7, 77, 3, 3, 1, 1, 1, sa.FILTER, 1.0), D),  # 72 slices
    ((1, 512, 7, 7, 33, 3, 3, 1, 1, 1, sa.FILTER, 1.0), {"path": {sa.CONV_DIRECT}, "ksplit": 8}),
    ((1, 704, 9, 8, 50, 3, 3, 1, 1, 2, sa.FILTER, 0.6), {"path": {sa.CONV_DIRECT}, "ksplit": 8}),  # runs of 352, split
]


@pytest.mark.parametrize("case,expect", CASES, ids=["x".join(str(v) for v in c[:10]) for c, _ in CASES])
def test_conv_direct_tiles(case, expect):
    conv_case(*case, seed=sum(case[:9]) + 5, dense_too=False, expect=expect)


def F(FM, TN, NP, WM):
    """The footprint kernel: 32*FM filters by 32*NP*TN pixels a tile, NP x WM wavefronts."""
    return {"path": {sa.CONV_FOOTPRINT}, "footprint_tile": (FM, TN, NP),
            "footprint_shape": (32 * NP * TN, 32 * FM, NP, WM)}


# the footprint kernel's shapes with several wavefronts over the filters of one
# input copy, or 64-pixel tiles: last tiles partly filled in filters and pixels,
# images that end within a tile, columns that are no whole step of 16.  At least
# 20 columns: the largest output of a layer with a few passes 10 times the RMS,
# where the rounding to bf16 alone (2^-9 of it) is past the bar of 2e-2.
FOOTPRINT = [
    ((1, 256, 17, 16, 9, 1, 1, 1, 0, 1, sa.SHAPE, 0.2), F(2, 1, 2, 2)),
    ((17, 512, 11, 10, 568, 1, 1, 1, 0, 2, sa.SHAPE, 0.1), F(4, 1, 2, 2)),
    ((33, 96, 17, 17, 223, 3, 3, 1, 1, 1, sa.SHAPE, 0.2), F(4, 1, 3, 2)),
    ((129, 128, 9, 10, 282, 1, 1, 1, 0, 1, sa.SHAPE, 0.2), F(6, 1, 3, 2)),
    ((65, 48, 17, 17, 816, 3, 3, 2, 1, 2, sa.SHAPE, 0.1), F(8, 1, 3, 2)),
    ((65, 128, 28, 28, 309, 1, 1, 2, 0, 1, sa.SHAPE, 0.3), F(12, 1, 3, 2)),
    ((17, 256, 28, 27, 611, 1, 1, 1, 0, 1, sa.SHAPE, 0.1), F(12, 1, 4, 2)),
    ((36, 192, 30, 29, 47, 1, 1, 1, 0, 1, sa.SHAPE, 0.2), F(2, 1, 4, 2)),  # more threads than weight chunks in a slice
]


@pytest.mark.parametrize("case,expect", FOOTPRINT, ids=["x".join(str(v) for v in c[:10]) for c, _ in FOOTPRINT])
def test_conv_footprint_tiles(case, expect):
    conv_case(*case, seed=sum(case[:9]) + 5, dense_too=False, expect=expect)
