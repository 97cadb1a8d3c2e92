"""The kernels behind a bf16 3x3 convolution, forward and input gradient, each at the sizes where it can go wrong: channels that fill
no tile or no step, more channel tiles than one block has wavefronts, pixels that end inside a tile, images narrower than the
window."""
import ctypes

import pytest

import harness
import paper_2408_08015_amd as lib
from asteroid_workloads import gen
from asteroid_workloads.configs import conv, simple
from test_parity_gpu import A, one_bf16  # noqa: F401  (A: the fixture)

GENERAL, HALO, RESIDENT = 0, 1, 2


def pick(B, h, w, cin, cout):
    """(groups of 32 pixels, wavefronts, blocks over the output channels) of the resident kernel, or None."""
    out = (ctypes.c_int * 3)()
    return tuple(out) if ctypes.CDLL(lib.lib_path()).ast_conv_res_choice(B, h, w, cin, cout, out) else None


# cin, cout, h, w, B
SIZES = [
    ((8, 8, 5, 5, 1), (1, 1, 1)),            # half a step of contracted channels, a quarter of a tile
    ((24, 40, 9, 7, 3), (1, 2, 1)),
    ((48, 96, 45, 45, 2), (1, 3, 1)),
    ((16, 264, 6, 11, 4), (1, 5, 2)),        # nine tiles in two blocks of five wavefronts
    ((520, 16, 4, 4, 3), (1, 1, 1)),         # more chunks in a row than a block has threads
    ((64, 64, 31, 33, 2), (1, 2, 1)),
    ((32, 64, 1, 1, 37), (1, 2, 1)),         # one-pixel images
    ((16, 32, 1, 50, 2), (1, 1, 1)),
    ((16, 32, 50, 1, 2), (1, 1, 1)),
    ((64, 128, 40, 40, 12), (2, 4, 1)),      # 64 pixels to a block
    ((24, 32, 60, 60, 20), (2, 1, 1)),
]


@pytest.mark.parametrize("sizes,want", SIZES)
def test_choice_of_the_resident_kernel(sizes, want):
    cin, cout, h, w, B = sizes
    assert pick(B, h, w, cin, cout) == want


def test_rows_too_long_for_the_resident_kernel():
    assert pick(1, 3, 1200, 64, 64) is None and pick(1, 3, 60, 640, 64) is None


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", [GENERAL, HALO, RESIDENT])
@pytest.mark.parametrize("sizes", [s[0] for s in SIZES])
def test_conv(A, monkeypatch, sizes, kernel):
    cin, cout, h, w, B = sizes
    if kernel == HALO and (cin % 64 or cout % 64):
        pytest.skip("whole slices of 64 channels only")
    if kernel == GENERAL and B * h * w > 10000:
        pytest.skip("the tiles of the general kernel do not depend on the number of pixels")
    monkeypatch.setenv("ASTEROID_CONV_KERNEL", str(kernel))
    # the second convolution's input gradient is masked by the ReLU between them
    layers = [conv(cin, cout, 3, 1, 1, bias=True), simple("relu"), conv(cout, cin, 3, 1, 1, bias=True)]
    cfg = one_bf16(layers, (cin, h, w), "nhwc", B=B, M=1)
    inp = gen.make_inputs(cfg, randomize_affine=True)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    # bf16 values in another order of fp32 additions: a result on the other side of a rounding, 4e-3 of it
    assert sc["r0.y"] <= 1e-2 and sc["r0.dx"] <= 2e-2
    for name, err in sc["r0.G_all"]:
        assert err <= 2e-2, (name, err)
