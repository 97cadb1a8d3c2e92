"""GPU parity at the sizes where a tile, a split or a dispatch rule of the kernels can go wrong: remainders, the
smallest and largest of a range, both sides of a rule.  Oracle and tolerances of test_parity_gpu.py (fp32: 1e-4 for
activations, 1e-3 for gradients; sums of a few thousand fp32 terms differ by about 1e-6)."""
import numpy as np
import pytest

import harness
from asteroid_workloads import gen
from asteroid_workloads.configs import bn, conv, simple
from test_conv_choices import DIRECT_FORMS, PRODUCT_FORMS, SPLIT_WGRAD, WGRAD, WGRAD_FORMS, choice
from test_parity_gpu import A, check, one  # noqa: F401  (A: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,k,stride,h,w,B", [
    (96, 40, 3, 1, 7, 7, 5),        # tiles across samples; 12 groups of channels over 8 shares of the contraction
    (136, 72, 3, 1, 4, 3, 9),       # several samples per tile, 17 groups: the last chunk has empty shares
    (64, 64, 3, 1, 20, 20, 8),      # eight shares of the contraction in both products
    (40, 32, 3, 1, 2, 130, 2),      # rows longer than a tile
    (8, 40, 3, 1, 3, 400, 1),       # rows too long for the staged kernels: the direct ones
    (8, 8, 3, 1, 2, 2600, 1),
    (128, 128, 3, 2, 14, 14, 3),    # parity classes of 49 pixels each
    (72, 96, 3, 2, 7, 9, 5),        # odd size: classes of different sizes
    (64, 72, 3, 2, 30, 62, 2),      # stride-2 rows
    (192, 136, 1, 2, 9, 7, 4),      # 1x1: three of four classes are zeros; ragged 64 x 64 weight-gradient tiles
    (256, 64, 1, 2, 14, 14, 2),
])
def test_dense_conv_tiles(A, cin, cout, k, stride, h, w, B):
    check(one([conv(cin, cout, k, stride, k // 2)], (cin, h, w), B=B), rounds=1)


@pytest.mark.parametrize("cin,cout,k,stride,h,w,B", [f[0] for f in PRODUCT_FORMS + WGRAD_FORMS + DIRECT_FORMS] + SPLIT_WGRAD)
def test_dense_conv_forms(A, cin, cout, k, stride, h, w, B):
    check(one([conv(cin, cout, k, stride, k // 2)], (cin, h, w), B=B, M=1), rounds=1)


@pytest.mark.parametrize("c,h,w,B", [
    (8, 27, 27, 13),    # planes of 729 words: five samples per block, 16 words per thread in flight
    (6, 67, 67, 3),     # 4489 words: two chunks per plane
    (5, 1, 3, 2900),    # 1365 samples per block
    (3, 1, 1, 9001),    # one-word planes
])
def test_batchnorm_planes_not_a_multiple_of_16_bytes(A, c, h, w, B):
    check(one([bn(c), simple("relu6")], (c, h, w), B=B), rounds=1)


# weight-gradient tiles per block (co x ci); the products' forms: test_split_products_gpu.py
@pytest.mark.parametrize("cin,cout,h,w,B,tiles", [
    (96, 128, 16, 16, 64, "2x1"),
    (56, 232, 14, 14, 77, "2x1"),   # ragged rows of both operands
    (528, 520, 7, 7, 16, "2x2"),    # ... 17 tiles of either
    (24, 144, 19, 20, 60, "1x1"),   # one tile of input channels
    (160, 40, 13, 14, 90, "2x1"),   # an odd number of tiles of input channels
    (64, 96, 14, 14, 130, "1x2"),   # ... of output channels
    (33, 264, 27, 27, 36, "1x2"),   # planes no multiple of 16 bytes
    (80, 72, 25, 25, 20, "2x1"),
    (80, 24, 9, 9, 200, "1x1"),
    (24, 80, 9, 9, 200, "1x1"),
    (256, 192, 7, 7, 43, "1x1"),    # steps across samples of 49
    (33, 65, 7, 7, 3, "1x1"),       # few blocks: two steps, rows past both edges
    (8, 8, 1, 1, 5, "1x1"),         # fewer pixels than a step
    (1024, 40, 7, 7, 2, "1x1"),     # product split over eight wavefronts: eight groups of 16 channels each
    (1032, 40, 7, 7, 2, "1x1"),     # nine each; the last wavefront has two
    (40, 2056, 5, 5, 2, "1x1"),     # over four in the input gradient, 33 each, the last 30
])
def test_pointwise_conv_tiles(A, cin, cout, h, w, B, tiles):
    import ctypes
    out = (ctypes.c_int * 3)()
    ctypes.CDLL(A.lib_path()).ast_pw_wgrad_choice(B, cin, cout, h * w, 2 ** 31 - 1, out)
    assert ("2x2", "2x1", "1x2", "1x1")[out[0]] == tiles
    check(one([conv(cin, cout, 1, 1, 0)], (cin, h, w), B=B), rounds=1)


@pytest.mark.parametrize("cin,cout,k,stride,hw,B", [
    (512, 2048, 1, 1, 7, 128),      # pointwise, 2x2 weight tiles: ranges of 25 steps
    (24, 144, 1, 1, 56, 128),       # 1x1 tiles, ranges of 31 steps
    (960, 160, 1, 1, 7, 512),       # 2x2 tiles, ranges of 31 steps
    (512, 512, 3, 1, 7, 128),       # dense
    (64, 64, 3, 1, 56, 64),
    (1024, 2048, 1, 2, 14, 128),    # 64 x 64 tiles
])
def test_rounding_of_weight_gradients_does_not_grow_with_the_micro_batch(A, cin, cout, k, stride, hw, B):
    """An fp32 addition rounds by 2^-25.3 of its result (root mean square), a chain of n additions of independent terms by
    sqrt(n / 2) as much of its sum.  No chain is longer than 128 pixels: 2.0e-7, and 0.3e-7 for the last roundings."""
    import torch
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    ho = (hw - 1) // stride + 1
    x = torch.randn(B, cin, hw, hw, generator=g, device=dev)
    dy = torch.randn(B, cout, ho, ho, generator=g, device=dev)
    y = torch.empty_like(dy)
    torch.cuda.synchronize()
    st = A.Stage([conv(cin, cout, k, stride, k // 2)], B, 1, 1, (cin, hw, hw), needs_input_grad=False)
    st.set_params(np.zeros(st.num_params, np.float32))
    st.forward(0, x, None, y)
    st.backward(0, dy)
    got = torch.from_numpy(st.get_grads()).to(dev).double().reshape(cout, cin, k, k)
    st.close()
    want = torch.zeros_like(got)
    xp = torch.nn.functional.pad(x, (k // 2,) * 4)
    rows = torch.empty(cout, B * ho * ho, dtype=torch.float64, device=dev)
    rows.copy_(dy.permute(1, 0, 2, 3).reshape(cout, -1))
    for u in range(k):
        for v in range(k):
            cols = xp[:, :, u:u + stride * (ho - 1) + 1:stride, v:v + stride * (ho - 1) + 1:stride]
            want[:, :, u, v] = rows @ cols.permute(0, 2, 3, 1).reshape(-1, cin).double()
    assert float((got - want).norm() / want.norm()) < 2.2e-7


@pytest.mark.parametrize("layers,shape,B", [
    ([conv(128, 128, 1, 1, 0)] * 2, (128, 28, 28), 32),   # pointwise: 192 partials a layer for speed, 48 here
    ([conv(64, 64, 3, 1, 1)] * 5, (64, 28, 28), 4),       # dense: 49 and 25
])
def test_partials_of_a_stage_that_just_fits_the_static_workspace(A, layers, shape, B):
    cfg = one(layers, shape, B=B, M=1)
    inp = gen.make_inputs(cfg, randomize_affine=True)
    ref, _, mem = harness.run_hip(cfg, inp, K=1, rounds=1)
    assert mem[3] <= 32 << 20
    got, _, _ = harness.run_hip(cfg, inp, K=1, rounds=1, static_backward=True)
    for k in ("y", "dx", "G", "W"):
        assert np.array_equal(ref[0][k], got[0][k]), k
    check(cfg, rounds=1)


@pytest.mark.parametrize("n,cin,cout,hw,k,staged", [
    (1400, 64, 64, 112, 1, False),   # x of 4.5 GB: beyond 32-bit offsets, direct kernels
    (1337, 128, 32, 56, 3, True),    # x of 2 146 729 984 bytes, the last that the staged kernels take
])
def test_strided_conv_of_a_tensor_around_the_offset_limit(A, n, cin, cout, hw, k, staged):
    """Three samples spread over the tensor are not zero: the gradients are those of these samples alone."""
    import torch
    assert (choice(WGRAD, n, cin, cout, hw, hw, k, 2) is not None) == staged
    dev, at, ho = torch.device("cuda:0"), [0, n // 2, n - 1], hw // 2
    g = torch.Generator().manual_seed(3)
    xs, ws = torch.randn(3, cin, hw, hw, generator=g), torch.randn(cout, cin, k, k, generator=g) / (cin * k * k) ** 0.5
    gs = torch.randn(3, cout, ho, ho, generator=g)
    x = torch.zeros(n, cin, hw, hw, device=dev)
    dy = torch.zeros(n, cout, ho, ho, device=dev)
    for i, s in enumerate(at):
        x[s].copy_(xs[i])
        dy[s].copy_(gs[i])
    y = torch.empty_like(dy)
    torch.cuda.synchronize()
    st = A.Stage([conv(cin, cout, k, 2, k // 2)], n, 1, 1, (cin, hw, hw), needs_input_grad=False)
    st.set_params(ws.numpy().ravel())
    st.forward(0, x, None, y)
    st.backward(0, dy)
    got = torch.from_numpy(st.get_grads()).reshape(ws.shape)
    st.close()
    wd = ws.double().requires_grad_()
    yd = torch.nn.functional.conv2d(xs.double(), wd, stride=2, padding=k // 2)
    yd.backward(gs.double())
    for have, want in ((got, wd.grad), (y[at].cpu(), yd.detach())):
        assert float((have.double() - want).norm() / want.norm()) < 1e-6   # sums of at most 9408 fp32 products
    assert not y[1:n // 2].any() and not y[n // 2 + 1:n - 1].any()
