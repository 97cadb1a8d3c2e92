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
    ((104, 104, 23, 31, 23), (2, 4, 1)),     # ... 15 pixels in the last one
    ((40, 72, 27, 57, 16), (2, 3, 1)),       # ... 48
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


def whole_numbers(A, sizes):
    """Two convolutions with a ReLU between them and a stage's output, in whole numbers whose sums stay below 2^24: the fp32
    sums are exact in any order, and what is stored is their one rounding to bf16.  Returns the launches by name."""
    import torch
    import torch.nn.functional as F
    cin, cout, h, w, B = sizes
    dev, g = torch.device("cuda:0"), torch.Generator().manual_seed(5)
    x, dy = (torch.randint(-1, 2, (B, h, w, cin), generator=g).float() for _ in range(2))
    w1, w2 = (torch.randint(-1, 2, (o, i, 3, 3), generator=g).float() for o, i in ((cout, cin), (cin, cout)))
    b1, b2 = (torch.randint(-4, 5, (o,), generator=g).float() for o in (cout, cin))
    st = A.Stage([conv(cin, cout, 3, 1, 1, bias=True), simple("relu"), conv(cout, cin, 3, 1, 1, bias=True)], B, 1, 1, (cin, h, w),
                 "bf16", "nhwc")
    st.set_params(torch.cat([t.flatten() for t in (w1, b1, w2, b2)]).numpy())
    xd, gd = x.to(dev, torch.bfloat16), dy.to(dev, torch.bfloat16)
    y, dx = torch.empty_like(xd), torch.empty_like(xd)
    torch.cuda.synchronize()
    st.profile_begin("conv")
    st.forward(0, xd, None, y)
    st.backward(0, gd, dx)
    names = st.profile_end()
    st.close()
    bf16 = lambda t: t.bfloat16().float()
    nchw = lambda t: t.permute(0, 3, 1, 2)
    a = bf16(F.conv2d(nchw(x), w1, b1, padding=1).relu())
    want_y = bf16(F.conv2d(a, w2, b2, padding=1))
    ga = bf16(F.conv_transpose2d(nchw(dy), w2, padding=1)) * (a > 0)
    want_dx = bf16(F.conv_transpose2d(ga, w1, padding=1))
    assert float(a.abs().max()) * 9 * cout < 1 << 24 and float(ga.abs().max()) * 9 * cout < 1 << 24
    assert torch.equal(nchw(y.float().cpu()), want_y)
    assert torch.equal(nchw(dx.float().cpu()), want_dx)
    return names


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [s[0] for s in SIZES])
def test_every_pixel_of_the_resident_kernel(A, monkeypatch, sizes):
    monkeypatch.setenv("ASTEROID_CONV_KERNEL", str(RESIDENT))
    names = whole_numbers(A, sizes)
    assert sum(n for name, (n, _) in names.items() if name.startswith("conv_res_kernel")) == 4


# where nothing is asked for: on either side of the lines between the halo and the resident kernel, the same both ways
@pytest.mark.gpu
@pytest.mark.parametrize("sizes,kernel", [
    ((64, 64, 42, 50, 20), "conv3x3_halo"), ((64, 64, 41, 51, 20), "conv_res"),
    ((192, 256, 40, 40, 20), "conv3x3_halo"), ((192, 192, 40, 39, 20), "conv_res"),
    ((256, 256, 50, 52, 10), "conv3x3_halo"), ((256, 256, 50, 51, 10), "conv_res"),
    ((72, 64, 45, 45, 22), None),              # whole slices of 64 contracted channels one way only
    ((64, 192, 52, 52, 16), None),             # 192 of 256 output channels one way
])
def test_kernel_by_size(A, monkeypatch, sizes, kernel):
    monkeypatch.delenv("ASTEROID_CONV_KERNEL", raising=False)
    count = {k: 0 for k in ("conv3x3_halo", "conv_res")}
    for name, (n, _) in whole_numbers(A, sizes).items():
        for k in count:
            count[k] += n if name.startswith(k) else 0
    want = {kernel: 4} if kernel else {"conv3x3_halo": 2, "conv_res": 2}
    assert {k: v for k, v in count.items() if v} == want
