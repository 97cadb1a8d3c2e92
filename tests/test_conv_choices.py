"""Which kernel a dense fp32 convolution runs on, at both sides of each limit (host code only)."""
import ctypes

import pytest

import paper_2408_08015_amd as A
from asteroid_workloads.configs import bn, conv, irb, simple

FWD, DGRAD, WGRAD, FEWER = 0, 1, 2, 3   # FEWER: a weight gradient whose stage has to fit the static workspace


def choice(what, n, cin, cout, h, w, k, s):
    """None: other kernels; else the words of the staged fp32 kernel's block shape."""
    out = (ctypes.c_int * 6)()
    lib = ctypes.CDLL(A.lib_path())
    return tuple(out) if lib.ast_conv_lds_choice(what, n, cin, cout, h, w, k, s, out) else None


def split_choice(what, n, cin, cout, h, w, k, s):
    """The same for the kernels on the bf16 matrix cores."""
    out = (ctypes.c_int * 6)()
    lib = ctypes.CDLL(A.lib_path())
    if what == WGRAD:
        return tuple(out) if lib.ast_conv_wgrad_x3_choice(n, cin, cout, h, w, k, s, out) else None
    return tuple(out) if lib.ast_conv_x3_choice(what, n, cin, cout, h, w, k, s, out) else None


# Sizes (cin, cout, k, stride, h, w, B) whose parity is checked on the GPU, each for the form that its choice must be, so
# that a change of the cost models cannot leave a form untested.
#   weight gradient: buffers, scratch areas of a flush inside a buffer, stages per block, stages per flush
WGRAD_FORMS = [
    ((40, 392, 3, 1, 6, 150, 3), (1, 2, 3, 2)),       # rows of 128 and more
    ((392, 392, 3, 2, 7, 7, 12), (2, 1, 3, 2)),       # stride 2
    ((40, 392, 3, 2, 28, 28, 12), (2, 2, 5, 3)),
    ((392, 392, 3, 2, 5, 90, 2), (1, 2, 3, 2)),
    ((72, 392, 1, 2, 14, 14, 24), (2, 1, 2, 2)),      # 1x1: 64 x 64 tiles
    ((72, 136, 1, 2, 6, 150, 12), (1, 2, 2, 2)),
]
#   ... of stride 1 and shorter rows: only where the stage has to fit the static workspace
FEWER_FORMS = [
    ((256, 392, 3, 1, 63, 8, 22), (2, 0, 25, 13)),    # flushes of unequal length, both scratch areas past the buffers
    ((192, 392, 3, 1, 34, 16, 13), (2, 1, 19, 7)),
    ((192, 512, 3, 1, 25, 8, 40), (2, 1, 8, 8)),      # no flush before the end
    ((192, 392, 3, 1, 9, 78, 10), (2, 2, 37, 13)),
    ((192, 392, 3, 1, 4, 98, 20), (1, 2, 21, 7)),
]
#   ... else these run on the bf16 matrix cores (their forms: test_split_products_gpu.py)
SPLIT_WGRAD = [(136, 392, 3, 1, 7, 7, 32), (40, 392, 3, 1, 14, 14, 12), (40, 264, 3, 1, 30, 62, 2), (40, 72, 3, 1, 5, 90, 12)]

#   products, forward and input gradient: 32-row tiles of result channels, groups of 32 pixels, shares of the contraction
PRODUCT_FORMS = [
    ((40, 40, 3, 1, 56, 56, 8), (2, 4, 1), (2, 4, 1)),
    ((264, 40, 3, 1, 5, 90, 12), (1, 2, 2), (2, 4, 1)),     # nine tiles: the last pair has one
    ((64, 264, 3, 1, 5, 90, 12), (2, 4, 2), (1, 2, 2)),     # ... and the sums of two shares
    ((64, 72, 3, 2, 15, 62, 12), (2, 1, 4), (1, 3, 4)),     # stride 2: classes of 1, 2 and 4 taps in the input gradient
    ((200, 64, 3, 2, 5, 90, 5), (1, 2, 2), (2, 2, 4)),
    ((264, 40, 3, 2, 5, 90, 12), (1, 2, 2), (2, 4, 1)),
    ((64, 264, 1, 2, 6, 150, 8), (2, 2, 4), (1, 2, 4)),     # 1x1 stride 2
    ((264, 64, 1, 2, 6, 150, 8), (1, 2, 4), (2, 2, 4)),
]
#   rows too long for the staged kernels: which of forward, input gradient and weight gradient are staged all the same
DIRECT_FORMS = [
    ((8, 40, 3, 1, 3, 400, 1), (False, False, False)),      # rows a multiple of 16 bytes
    ((8, 40, 3, 1, 3, 401, 2), (False, False, False)),
    ((8, 40, 3, 2, 3, 400, 1), (False, True, False)),
    ((8, 40, 3, 2, 3, 401, 2), (False, True, False)),
    ((24, 40, 3, 2, 3, 2601, 2), (False, False, False)),
    ((8, 40, 1, 2, 3, 401, 2), (True, True, False)),
    ((40, 24, 1, 2, 3, 2601, 2), (False, False, False)),
    ((40, 8, 1, 2, 4, 802, 1), (False, False, False)),
]


@pytest.mark.parametrize("sizes,forward,backward", PRODUCT_FORMS)
def test_form_of_the_staged_products(sizes, forward, backward):
    cin, cout, k, s, h, w, n = sizes
    for what, want in ((FWD, forward), (DGRAD, backward)):
        got = choice(what, n, cin, cout, h, w, k, s)
        assert got is not None and got[:3] == want


@pytest.mark.parametrize("sizes,staged", DIRECT_FORMS)
def test_rows_too_long_for_the_staged_kernels(sizes, staged):
    cin, cout, k, s, h, w, n = sizes
    assert tuple(choice(what, n, cin, cout, h, w, k, s) is not None for what in (FWD, DGRAD, WGRAD)) == staged


@pytest.mark.parametrize("what,sizes,want", [(WGRAD,) + f for f in WGRAD_FORMS] + [(FEWER,) + f for f in FEWER_FORMS])
def test_form_of_the_staged_weight_gradient(what, sizes, want):
    cin, cout, k, s, h, w, n = sizes
    got = choice(what, n, cin, cout, h, w, k, s)
    assert got is not None and (got[3], got[5], got[1], got[4]) == want
    assert (split_choice(WGRAD, n, cin, cout, h, w, k, s) is not None) == (what == FEWER)


@pytest.mark.parametrize("cin,cout,k,s,h,w,n", SPLIT_WGRAD)
def test_weight_gradients_on_the_bf16_matrix_cores(cin, cout, k, s, h, w, n):
    assert choice(WGRAD, n, cin, cout, h, w, k, s) is None and split_choice(WGRAD, n, cin, cout, h, w, k, s) is not None


@pytest.mark.parametrize("what", [FWD, DGRAD, WGRAD])
@pytest.mark.parametrize("n,cin,cout,h,k,s,reads_x,reads_g", [
    # the kernels that stage through LDS, fp32 or split, address a tensor with 32-bit byte offsets below 2 GiB
    (668, 64, 64, 112, 1, 2, True, True),       # x of 2 145 124 352 bytes
    (669, 64, 64, 112, 1, 2, False, True),      # x of 2 148 335 616
    (1400, 64, 64, 112, 1, 2, False, True),     # x of 4.5 GB, and the subsampled x of 1.1 GB
    (2674, 64, 64, 112, 1, 2, False, True),
    (2675, 64, 64, 112, 1, 2, False, False),    # dy of 2 147 532 800
    (329, 128, 128, 56, 3, 2, True, True),      # x of 528 MB
    (1337, 128, 128, 56, 3, 2, True, True),     # x of 2 146 729 984
    (1338, 128, 128, 56, 3, 2, False, True),
    (2674, 64, 64, 56, 3, 1, True, True),
    (2675, 64, 64, 56, 3, 1, False, False),     # x and dy of 2 147 532 800
    (167, 8, 1024, 56, 3, 1, True, True),
    (168, 8, 1024, 56, 3, 1, True, False),      # dy of 2 157 969 408, x of 16 MB
])
def test_size_limit_of_the_staged_convolutions(what, n, cin, cout, h, k, s, reads_x, reads_g):
    assert (n * cin * h * h * 4 < 2 ** 31) == reads_x
    assert (n * cout * ((h - 1) // s + 1) ** 2 * 4 < 2 ** 31) == reads_g
    want = {FWD: reads_x, DGRAD: reads_g, WGRAD: reads_x and reads_g}[what]
    staged, split = (c(what, n, cin, cout, h, h, k, s) is not None for c in (choice, split_choice))
    assert (staged or split) == want and not (staged and split)


# Stages whose workspace with the counts that are fastest is past the static scratch array (33.6 MB), and with fewer is not:
# backward_static takes them.
BN_PAIR = lambda c, m: [conv(c, m, 1), bn(m), simple("relu6"), conv(m, c, 1), bn(c)]
FIT_WITH_FEWER = [
    ([conv(64, 128, 1), simple("relu"), conv(128, 64, 1)], 64, 40, 16),     # one pointwise weight gradient is enough
    ([conv(256, 192, 1), simple("relu"), conv(192, 256, 1)], 256, 54, 5),
    (BN_PAIR(16, 384), 16, 18, 29),                                         # statistics partials as well
    (BN_PAIR(48, 64), 48, 32, 37),
    ([conv(64, 384, 3, 1, 1), bn(384), simple("relu")], 64, 35, 11),        # dense weight gradients
    ([conv(256, 144, 3, 1, 1), bn(144), simple("relu")], 256, 45, 17),
    (irb(8, 24, 1, 6), 8, 36, 28),
    (irb(128, 16, 1, 6), 128, 12, 14),
]


@pytest.mark.parametrize("layers,c,hw,n", FIT_WITH_FEWER)
def test_workspace_fits_the_static_array(layers, c, hw, n):
    assert A.plan_memory(layers, n, 1, 1, (c, hw, hw))[3] <= 32 << 20


def test_weight_gradient_ranges():
    """Chains of additions: at most 32 steps of 64 pixels to a range, or 64-bit sums in between."""
    lib = ctypes.CDLL(A.lib_path())
    out = (ctypes.c_int * 3)()
    for cin, cout, hw, n in ((512, 512, 3136, 22), (1024, 96, 3025, 60), (2048, 32, 3136, 85), (24, 144, 3136, 128)):
        steps = -(-n * hw // 64)
        lib.ast_pw_wgrad_choice(n, cin, cout, hw, 2 ** 31 - 1, out)
        assert not out[2] and -(-steps // out[1]) <= 32
        lib.ast_pw_wgrad_choice(n, cin, cout, hw, 5, out)
        assert out[2] and out[1] == 5 and out[0] != 0   # (not the block shape that has no registers left)


# Four row tiles: two groups of 32 pixels to a wavefront where that takes fewer rounds of blocks than one (three blocks of one group
# run on a compute unit, one of two), at sizes on either side of a whole round
@pytest.mark.parametrize("sizes,groups", [
    ((64, 128, 3, 1, 28, 28, 32), 2), ((64, 128, 3, 1, 28, 28, 31), 1),     # 784 blocks of one group; 760
    ((64, 256, 3, 1, 36, 36, 12), 2), ((64, 256, 3, 1, 36, 36, 13), 1),     # 244 blocks of two groups; 264
    ((128, 512, 3, 1, 14, 14, 41), 2), ((128, 512, 3, 1, 14, 14, 44), 1),   # 252; 272
    ((96, 384, 3, 1, 28, 28, 15), 1), ((64, 384, 3, 1, 20, 20, 33), 1),     # 276; 312: a second round that is nearly empty
    ((256, 384, 3, 1, 14, 14, 22), 2),                                      # two shares: 204 blocks of two groups for 405
    ((256, 160, 3, 1, 20, 20, 24), 1),                                      # ... 300 for 600: two rounds for three
    ((32, 128, 3, 1, 56, 56, 32), 4),
])
def test_pixel_groups_by_rounds(sizes, groups):
    cin, cout, k, s, h, w, B = sizes
    assert split_choice(FWD, B, cin, cout, h, w, k, s)[:2] == (groups, 4)
