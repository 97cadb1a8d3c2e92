"""GPU parity at the sizes where a tile, a split or a dispatch rule of the kernels can go wrong: remainders, the
smallest and largest of a range, both sides of a rule.  Oracle and tolerances of test_parity_gpu.py (fp32: 1e-4 for
activations, 1e-3 for gradients; sums of a few thousand fp32 terms differ by about 1e-6)."""
import pytest

from asteroid_workloads.configs import bn, conv, simple
from test_parity_gpu import A, check, one  # noqa: F401  (A: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,k,stride,h,w,B", [
    (96, 40, 3, 1, 7, 7, 5),        # tiles across samples; 12 groups of channels over 8 shares of the contraction
    (136, 72, 3, 1, 4, 3, 9),       # several samples per tile, 17 groups: the last chunk has empty shares
    (64, 64, 3, 1, 20, 20, 8),      # two channel tiles per wavefront
    (40, 32, 3, 1, 2, 130, 2),      # rows longer than a tile
    (8, 40, 3, 1, 3, 400, 1),       # rows too long for the staged weight gradient
    (8, 8, 3, 1, 2, 2600, 1),       # ... and for the staged product: the direct kernels
    (128, 128, 3, 2, 14, 14, 3),    # parity classes of 49 pixels each
    (72, 96, 3, 2, 7, 9, 5),        # odd size: classes of different sizes
    (64, 72, 3, 2, 30, 62, 2),      # stride-2 rows, single-buffered weight gradient
    (192, 136, 1, 2, 9, 7, 4),      # 1x1: three of four classes are zeros; ragged 64 x 64 weight-gradient tiles
    (256, 64, 1, 2, 14, 14, 2),
])
def test_dense_conv_tiles(A, cin, cout, k, stride, h, w, B):
    check(one([conv(cin, cout, k, stride, k // 2)], (cin, h, w), B=B), rounds=1)


@pytest.mark.parametrize("c,h,w,B", [
    (8, 27, 27, 13),    # planes of 729 words: five samples per block, 16 words per thread in flight
    (6, 67, 67, 3),     # 4489 words: two chunks per plane
    (5, 1, 3, 2900),    # 1365 samples per block
    (3, 1, 1, 9001),    # one-word planes
])
def test_batchnorm_planes_not_a_multiple_of_16_bytes(A, c, h, w, B):
    check(one([bn(c), simple("relu6")], (c, h, w), B=B), rounds=1)
