"""fp32 products on the bf16 matrix cores with their operands split in three: the kernel forms at sizes on either side of
their rules, their rounding error, and operands that are not finite."""
import numpy as np
import pytest

import harness
from asteroid_workloads import gen
from asteroid_workloads.configs import bn, conv, simple
from test_conv_choices import FEWER_FORMS
from test_parity_gpu import A, one  # noqa: F401  (A: the fixture)

pytestmark = pytest.mark.gpu

# Relative error of a product of normal matrices: at most 2^-24 from the last rounding, 2^-24 from the five small products, and
# a random walk of one rounding per 8 terms, of which each is 2^-25.3 of the sum so far (root mean square): K / 8 of them are
# 2^-25.3 * sqrt(K / 16) of the whole sum, and the bound has 2^-24 there.  The fp32 matrix instructions, which round every
# second term, are at twice that walk.  Weight gradients: chains of at most 64 roundings, 2^-25.3 * sqrt(32) = 1.4e-7, and
# 0.6e-7 for the last roundings; 1e-7 measured.
BOUND_W = 2e-7


def bound(k):
    return 1.2e-7 + 2.0 ** -24 * (k / 16) ** 0.5


# Forms of a pointwise product: pixels per lane x row tiles of a wavefront, a contraction split over four or eight
# wavefronts, all row tiles in one wavefront
PX1, PX1X2, PX2, PX2X2, KS4, KS4X2, KS8, WIDE, FAR = range(9)


def pw_choice(dgrad, n, cin, cout, hw):
    import ctypes
    out = (ctypes.c_int * 4)()
    import paper_2408_08015_amd as A_
    ctypes.CDLL(A_.lib_path()).ast_pw_choice(dgrad, n, cin, cout, hw, out)
    return out[0]


POINTWISE = [
    (15, 33, 5, 7, 3, PX1, PX1),            # one group of 16 channels, odd planes, a second row tile of one row
    (17, 31, 9, 9, 2, PX1, PX1),
    (96, 576, 14, 14, 1, KS4, KS4),         # six groups of channels in four shares
    (576, 96, 7, 7, 2, KS8, KS4),
    (528, 264, 7, 7, 10, KS8, KS4),         # 33 groups in eight shares; 17 in four
    (528, 520, 7, 7, 16, KS4X2, KS4X2),     # two row tiles each, the last pair has one
    (1032, 392, 7, 7, 20, KS4X2, KS4),
    (81, 40, 25, 24, 32, PX2, PX1),         # 600 pixels a plane
    (80, 72, 24, 24, 90, PX2, PX2),
    (104, 136, 24, 24, 35, PX2, PX2),       # five row tiles
    (104, 200, 24, 24, 25, PX2X2, PX2),     # seven: the last pair has one
    (200, 200, 24, 26, 25, PX2X2, PX2X2),
    (80, 72, 25, 25, 20, PX1X2, PX1X2),     # odd planes; three row tiles
    (16, 104, 56, 56, 20, WIDE, PX2),       # all row tiles in one wavefront
    (33, 264, 28, 28, 36, WIDE, PX2),       # ... nine tiles in two shares
    (64, 96, 56, 56, 24, WIDE, PX2X2),
    (40, 40, 1, 3, 70, PX1, PX1),           # planes of three pixels: a wavefront spans a dozen samples
]


@pytest.mark.parametrize("cin,cout,h,w,B,fwd,dgrad", POINTWISE)
def test_pointwise_forms(A, cin, cout, h, w, B, fwd, dgrad):
    assert (pw_choice(0, B, cin, cout, h * w), pw_choice(1, B, cin, cout, h * w)) == (fwd, dgrad)
    cfg = one([conv(cin, cout, 1)], (cin, h, w), B=B, M=1)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    assert sc["r0.y"] <= bound(cin)
    assert sc["r0.dx"] <= bound(cout)
    assert harness.rel_l2(hip[0]["G"], ora[0]["G"]) <= BOUND_W


@pytest.mark.parametrize("cin,cout,k,s,h,B", [(2048, 64, 1, 1, 28, 12), (1024, 256, 1, 1, 14, 8), (512, 2048, 1, 1, 7, 8),
                                              (64, 256, 1, 1, 56, 8), (512, 64, 3, 1, 14, 30), (32, 512, 3, 1, 40, 8),
                                              (512, 128, 1, 2, 28, 8)])
def test_rounding_of_operands_of_one_sign(A, cin, cout, k, s, h, B):
    """Every partial sum of positive operands is rounded in the same binade again and again: with a rounding that goes to one
    side, the errors of the steps of 16 terms would add up (half a step's 2^-24 each: 2e-6 at 2048 channels) and show as a
    mean; to nearest they are the random walk of the bound above."""
    import torch
    gen_ = torch.Generator(device="cuda")
    gen_.manual_seed(4)
    r = lambda *a: torch.randn(*a, generator=gen_, device="cuda").abs_()
    ho = (h - 1) // s + 1
    x, g, w = r(B, cin, h, h), r(B, cout, ho, ho), r(cout, cin, k, k)
    st = A.Stage([conv(cin, cout, k, s, k // 2)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    st.set_params(w.cpu().numpy().ravel())
    y, dx = torch.empty_like(g), torch.empty_like(x)
    st.forward(0, x, None, y, None)
    st.backward(0, g, dx)
    G = torch.from_numpy(st.get_grads()).cuda().view(w.shape)
    st.close()
    p = k // 2
    xp = torch.nn.functional.pad(x.double(), (p, p, p, p))
    ry, rdx, rG = torch.zeros(cout, B * ho * ho, dtype=torch.float64, device="cuda"), torch.zeros_like(xp), torch.zeros_like(w).double()
    gm = g.double().permute(1, 0, 2, 3).reshape(cout, -1).contiguous()
    for u in range(k):
        for v in range(k):
            sl = (slice(None), slice(None), slice(u, u + s * (ho - 1) + 1, s), slice(v, v + s * (ho - 1) + 1, s))
            xs, wt = xp[sl].permute(1, 0, 2, 3).reshape(cin, -1).contiguous(), w[:, :, u, v].double().contiguous()
            ry += wt @ xs
            rdx[sl] += (wt.t().contiguous() @ gm).view(cin, B, ho, ho).permute(1, 0, 2, 3)
            rG[:, :, u, v] = gm @ xs.t().contiguous()
    ry, rdx = ry.view(cout, B, ho, ho).permute(1, 0, 2, 3), rdx[:, :, p:p + h, p:p + h]
    for got, want, lim in ((y, ry, bound(cin * k * k)), (dx, rdx, bound(cout * k * k)), (G, rG, BOUND_W)):
        d = got.double() - want
        assert float(d.norm() / want.norm()) <= lim
        assert abs(float(d.mean() / want.mean())) <= 2e-8


def test_pointwise_skip_gradient(A):
    # the input gradient of a block's first convolution takes the skip gradient in its epilogue: few and many row tiles
    for cin, mid, hw, B in ((96, 24, 56, 28), (24, 40, 12, 3), (160, 200, 7, 2)):
        layers = [simple("res_begin"), conv(cin, mid, 1), conv(mid, cin, 1), simple("res_add")]
        cfg = one(layers, (cin, hw, hw), B=B, M=1)
        inp = gen.make_inputs(cfg)
        ora, _ = harness.run_oracle(cfg, inp, rounds=1)
        hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
        sc = harness.score(cfg, hip, ora)
        assert max(sc["r0.y"], sc["r0.dx"]) <= 4e-7


@pytest.mark.parametrize("cin,cout,h,B,fwd,dgrad", [
    (24, 40, 6, 3, PX1, PX1), (272, 40, 7, 2, KS8, PX1), (40, 272, 7, 2, PX1, KS4), (528, 520, 7, 16, KS4X2, KS4X2),
    (72, 72, 24, 90, PX2, PX2), (80, 72, 25, 20, PX1X2, PX1X2), (104, 200, 24, 25, PX2X2, PX2), (24, 104, 56, 20, WIDE, PX2)])
def test_pointwise_operands_that_are_not_finite(A, cin, cout, h, B, fwd, dgrad):
    """An infinity or NaN reaches the outputs that its definition gives and no others, with the right sign, and the largest
    finite values are still values."""
    import torch
    assert (pw_choice(0, B, cin, cout, h * h), pw_choice(1, B, cin, cout, h * h)) == (fwd, dgrad)
    rng = np.random.default_rng(3)
    x = rng.standard_normal((B, cin, h, h)).astype(np.float32)
    dy = rng.standard_normal((B, cout, h, h)).astype(np.float32)
    wt = rng.standard_normal((cout, cin)).astype(np.float32)
    big = np.float32(3.4e38)   # rounds to infinity in bf16
    x[0, 1, 0, 0] = np.inf
    x[0, 2, 1, 1] = np.nan
    x[0, :, 2, 2] = 0
    x[0, 3, 2, 2] = big
    wt[:, 3] *= 1e-3
    dy[B - 1, 5, 0, 1] = -np.inf
    st = A.Stage([conv(cin, cout, 1)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    st.set_params(wt.ravel())
    dev = torch.device("cuda:0")
    tx, tg = torch.from_numpy(x).to(dev), torch.from_numpy(dy).to(dev)
    y, dx = torch.empty_like(tg), torch.empty_like(tx)
    st.forward(0, tx, None, y, None)
    st.backward(0, tg, dx)
    torch.cuda.synchronize()
    G = st.get_grads().reshape(cout, cin)
    st.close()
    with np.errstate(all="ignore"):
        ref = lambda a, b: np.matmul(a.astype(np.float64), b.astype(np.float64)).astype(np.float32)
        ry = ref(wt, x.reshape(B, cin, -1)).reshape(dy.shape)
        rdx = ref(wt.T, dy.reshape(B, cout, -1)).reshape(x.shape)
        rG = np.zeros((cout, cin), np.float32)
        for n in range(B):
            rG = rG + ref(dy[n].reshape(cout, -1), x[n].reshape(cin, -1).T)
    for got, want in ((y.cpu().numpy(), ry), (dx.cpu().numpy(), rdx), (G, rG)):
        fin = np.isfinite(want)
        assert not fin.all()
        np.testing.assert_array_equal(got[~fin], want[~fin])
        assert np.isfinite(got[fin]).all()
        np.testing.assert_allclose(got[fin], want[fin], rtol=1e-5, atol=2e-3)


@pytest.mark.parametrize("cin,cout,h,B,form", [(24, 104, 56, 20, WIDE), (104, 200, 24, 25, PX2X2), (16, 40, 14, 9, PX1)])
def test_statistics_of_operands_that_round_to_infinity(A, cin, cout, h, B, form):
    """The sums that a product leaves for the BatchNorm behind it are those of the values it stored."""
    import torch
    assert pw_choice(0, B, cin, cout, h * h) == form
    rng = np.random.default_rng(8)
    x = rng.standard_normal((B, cin, h, h)).astype(np.float32)
    wt = rng.standard_normal((cout, cin)).astype(np.float32)
    x[B - 1, 3, 1, 2] = 3.4e38
    wt[:, 3] *= 1e-30            # (a value of 2^-110 is 8e-34; of smaller ones the pieces lose what lies under 2^-133)
    wt[1, 3] = 0                 # (a channel of ordinary values)
    st = A.Stage([conv(cin, cout, 1), bn(cout)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    st.set_params(np.concatenate([wt.ravel(), np.ones(cout, np.float32), np.zeros(cout, np.float32)]))
    y = torch.empty(B, cout, h, h, device="cuda")
    st.forward(0, torch.from_numpy(x).cuda(), None, y, None)
    torch.cuda.synchronize()
    st.close()
    z = np.matmul(wt.astype(np.float64), x.reshape(B, cin, -1).astype(np.float64))
    want = (z - z.mean((0, 2), keepdims=True)) / np.sqrt(z.var((0, 2), keepdims=True) + 1e-5)
    # (the values other than the large one are differences from the mean that it dominates)
    np.testing.assert_allclose(y.cpu().numpy().reshape(z.shape), want, rtol=1e-5, atol=2e-5)


@pytest.mark.parametrize("cin,cout,k,h,B", [(24, 144, 1, 56, 8), (256, 64, 1, 56, 4), (528, 520, 1, 7, 16), (512, 40, 1, 7, 4),
                                            (64, 64, 3, 56, 4), (256, 256, 3, 14, 2), (64, 64, 3, 56, 16)])
def test_time_of_operands_that_are_not_finite(A, cin, cout, k, h, B):
    """A mini-batch that has diverged takes a few times as long as another one, not a hundred times."""
    import torch
    st = A.Stage([conv(cin, cout, k, 1, k // 2)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    x, g = torch.randn(B, cin, h, h, device="cuda"), torch.randn(B, cout, h, h, device="cuda")
    y, dx = torch.empty_like(g), torch.empty_like(x)
    best = []
    for bad in (False, True):
        if bad:
            x.fill_(float("nan"))
            g.fill_(float("nan"))
        ts = []
        for _ in range(10):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda.synchronize()
            ev[0].record()
            st.forward(0, x, None, y, None)
            st.backward(0, g, dx)
            ev[1].record()
            torch.cuda.synchronize()
            st.step(0.0, 0.0)
            ts.append(ev[0].elapsed_time(ev[1]))
        best.append(min(ts))
    print("%d -> %d k%d %dx%d B %d: finite %.0f us, NaN %.0f us" % (cin, cout, k, h, h, B, 1e3 * best[0], 1e3 * best[1]))
    st.close()
    # (2.7 times the matrix instructions, on top of the first attempt, and loads that nothing hides)
    assert best[1] <= 8 * best[0]
    assert torch.isnan(y).all() and torch.isnan(dx).all()


def x3_choice(dgrad, n, cin, cout, h, w, k, s):
    import ctypes
    out = (ctypes.c_int * 6)()
    import paper_2408_08015_amd as A_
    lib = ctypes.CDLL(A_.lib_path())
    return tuple(out) if lib.ast_conv_x3_choice(dgrad, n, cin, cout, h, w, k, s, out) else None


# dense convolutions (cin, cout, k, stride, h, w, B), and the forms of forward and input gradient: groups of 32 pixels per
# wavefront, row tiles, pixel groups, shares of the contraction
DENSE = [
    ((32, 512, 3, 1, 40, 41, 8), (4, 4, 1, 1), (1, 1, 4, 2)),      # four pixel groups, forward
    ((512, 16, 3, 1, 40, 41, 8), None, (4, 4, 1, 1)),              # ... and back
    ((16, 64, 3, 1, 56, 56, 32), (4, 2, 4, 1), None),              # ... beside each other, as in a ResNet's first group
    ((32, 128, 1, 2, 111, 112, 8), (2, 4, 1, 1), (1, 1, 4, 1)),    # two: large strided 1x1
    ((64, 96, 3, 1, 9, 30, 20), (1, 3, 1, 2), (1, 2, 1, 2)),       # three row tiles; 270 pixels a plane
    ((32, 32, 3, 1, 5, 3, 3), (1, 1, 8, 1), (1, 1, 8, 1)),         # one tile, most of it past the last pixel
    ((128, 64, 3, 1, 7, 7, 2), (1, 2, 1, 4), (1, 4, 1, 2)),        # tiles across samples
    ((192, 32, 3, 1, 2, 63, 3), (1, 1, 8, 1), (1, 4, 1, 1)),       # rows of 63: no room for more shares
    ((64, 64, 3, 2, 15, 14, 3), (1, 2, 1, 2), (1, 2, 1, 2)),       # classes of different sizes
    ((160, 96, 3, 2, 8, 9, 2), (1, 2, 1, 2), (1, 4, 1, 2)),
    ((64, 128, 1, 2, 14, 14, 3), (1, 4, 1, 2), (1, 2, 1, 4)),      # 1x1: three of four classes are zeros
    ((512, 512, 3, 1, 7, 7, 3), (1, 1, 1, 8), (1, 1, 1, 8)),
    ((48, 64, 3, 1, 11, 11, 2), (1, 2, 4, 1), None),               # forward alone: 48 is no multiple of 32
    ((16, 128, 3, 1, 39, 39, 16), (2, 4, 2, 1), None),             # two pixel groups for four row tiles: 24336 pixels
    ((16, 128, 3, 1, 38, 39, 16), (1, 4, 1, 1), None),             # ... and one, of 23712
    ((256, 128, 3, 1, 20, 31, 20), (2, 4, 1, 2), (2, 4, 2, 1)),    # ... beside two shares of the contraction
]


@pytest.mark.parametrize("sizes,fwd,dgrad", DENSE)
def test_dense_forms(A, sizes, fwd, dgrad):
    cin, cout, k, s, h, w, B = sizes
    for d, want in ((0, fwd), (1, dgrad)):
        got = x3_choice(d, B, cin, cout, h, w, k, s)
        assert (got is not None) == (((cout, cin)[d] % 32, (cin, cout)[d] % 16) == (0, 0))
        assert (got[:4] if got else None) == want
    cfg = one([conv(cin, cout, k, s, k // 2)], (cin, h, w), B=B, M=1)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    assert sc["r0.y"] <= bound(cin * k * k)
    assert sc["r0.dx"] <= (bound(cout * k * k) if dgrad else 1e-6)


@pytest.mark.parametrize("cin,cout,k,s,h,B", [(64, 64, 3, 1, 12, 4), (64, 32, 3, 2, 9, 2), (256, 64, 3, 1, 5, 2),
                                              (32, 512, 3, 1, 41, 8)])   # (the last: four pixel groups per wavefront)
def test_dense_operands_that_are_not_finite(A, cin, cout, k, s, h, B):
    import torch
    rng = np.random.default_rng(4)
    ho = (h - 1) // s + 1
    x = rng.standard_normal((B, cin, h, h)).astype(np.float32)
    dy = rng.standard_normal((B, cout, ho, ho)).astype(np.float32)
    wt = (rng.standard_normal((cout, cin, k, k)) * 0.1).astype(np.float32)
    x[0, 1, 2, 2] = np.inf
    x[1, 5, 0, 3] = np.nan
    x[1, 7, h - 1, 0] = 3.4e38   # rounds to infinity in bf16
    wt[:, 7] *= 1e-6
    dy[0, 3, 1, 1] = -np.inf
    st = A.Stage([conv(cin, cout, k, s, k // 2)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    st.set_params(wt.ravel())
    dev = torch.device("cuda:0")
    tx, tg = torch.from_numpy(x).to(dev), torch.from_numpy(dy).to(dev)
    y, dx = torch.empty_like(tg), torch.empty_like(tx)
    st.forward(0, tx, None, y, None)
    st.backward(0, tg, dx)
    torch.cuda.synchronize()
    st.close()
    with np.errstate(all="ignore"):
        ry, rdx = np.zeros(dy.shape), np.zeros((B, cin, h + 2, h + 2))
        xp = np.zeros((B, cin, h + 2, h + 2))
        xp[:, :, 1:-1, 1:-1] = x
        for u in range(k):
            for v in range(k):
                # (only the taps inside the image: an infinity times the zero border is no term)
                sl = (slice(None), slice(None), slice(u, u + s * (ho - 1) + 1, s), slice(v, v + s * (ho - 1) + 1, s))
                ry += np.einsum("oc,ncij->noij", wt[:, :, u, v].astype(np.float64), xp[sl])
                rdx[sl] += np.einsum("oc,noij->ncij", wt[:, :, u, v].astype(np.float64), dy.astype(np.float64))
        rdx = rdx[:, :, 1:-1, 1:-1]
    for got, want in ((y.cpu().numpy(), ry.astype(np.float32)), (dx.cpu().numpy(), rdx.astype(np.float32))):
        fin = np.isfinite(want)
        assert not fin.all()
        np.testing.assert_array_equal(got[~fin], want[~fin])
        assert np.isfinite(got[fin]).all()
        big = np.abs(want) > 1e6
        np.testing.assert_allclose(got[fin & ~big], want[fin & ~big], rtol=1e-5, atol=1e-4)
        np.testing.assert_allclose(got[fin & big], want[fin & big], rtol=1e-5)


def wgrad_choice(n, cin, cout, h, w, k, s):
    import ctypes
    out = (ctypes.c_int * 4)()
    import paper_2408_08015_amd as A_
    lib = ctypes.CDLL(A_.lib_path())
    return tuple(out) if lib.ast_conv_wgrad_x3_choice(n, cin, cout, h, w, k, s, out) else None


def weight_gradient(A, x, dy):
    """Of the HIP path, and in 64 bits (terms inside the image alone)."""
    import torch
    (B, cin, h, w), cout = x.shape, dy.shape[1]
    st = A.Stage([conv(cin, cout, 3, 1, 1)], B, 1, 1, (cin, h, w), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    st.set_params(np.zeros(cout * cin * 9, np.float32))
    tx, tg = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
    y, dx = torch.empty_like(tg), torch.empty_like(tx)
    st.forward(0, tx, None, y, None)
    st.backward(0, tg, dx)
    torch.cuda.synchronize()
    G = st.get_grads().reshape(cout, cin, 3, 3)
    st.close()
    ref = np.zeros((cout, cin, 3, 3))
    x, dy = x.astype(np.float64), dy.astype(np.float64)
    with np.errstate(all="ignore"):
        for u in range(3):
            for v in range(3):
                gs = dy[:, :, max(0, 1 - u):h - max(0, u - 1), max(0, 1 - v):w - max(0, v - 1)]
                xs = x[:, :, max(0, u - 1):h - max(0, 1 - u), max(0, v - 1):w - max(0, 1 - v)]
                if gs.size:
                    ref[:, :, u, v] = (gs.transpose(1, 0, 2, 3).reshape(cout, -1) @ xs.transpose(1, 0, 2, 3).reshape(cin, -1).T)
    return G, ref


# (cin, cout, h, w, B), rows per stage, chunks of eight columns per row; loads of four, two and one words
WEIGHT_GRADIENTS = [
    ((8, 8, 1, 1, 1), 2, 1),           # one pixel
    ((33, 65, 3, 2, 1), 4, 1),         # tiles with one channel
    ((64, 96, 7, 7, 40), 8, 1),        # a sample per stage
    ((40, 72, 17, 23, 5), 2, 3),       # an odd number of chunks per row
    ((32, 32, 5, 48, 3), 1, 7),        # ... and per stage; rows of whole vectors
    ((64, 64, 30, 54, 9), 1, 7),
    ((64, 32, 40, 56, 8), 1, 8),       # runs of several stages: the ring goes round
    ((264, 264, 14, 13, 4), 4, 2),
    ((8, 40, 3, 63, 2), 1, 8),
    ((8, 40, 20, 64, 12), 1, 9),       # the long-row form
    ((16, 24, 9, 71, 7), 1, 9),
    ((8, 24, 12, 127, 5), 1, 16),
]


@pytest.mark.parametrize("sizes,rows,chunks", WEIGHT_GRADIENTS)
def test_dense_weight_gradient_forms(A, sizes, rows, chunks):
    cin, cout, h, w, B = sizes
    got = wgrad_choice(B, cin, cout, h, w, 3, 1)
    assert got is not None and got[:2] == (rows, chunks)
    assert wgrad_choice(B, cin, cout, h, w, 3, 2) is None and wgrad_choice(B, cin, cout, h, 128, 3, 1) is None
    rng = np.random.default_rng(5)
    x = rng.standard_normal((B, cin, h, w)).astype(np.float32)
    G, ref = weight_gradient(A, x, rng.standard_normal((B, cout, h, w)).astype(np.float32))
    # a sum in a wavefront is rounded at most 64 times, whose errors (2^-25.3 of the sum so far each) add up to less than
    # 2^-24 * sqrt(32) of it; one more of the sum of the wavefronts and of the partials each, and of the pieces
    assert np.linalg.norm(G - ref) <= 2.0 ** -24 * (32 ** 0.5 + 3) * np.linalg.norm(ref)


@pytest.mark.parametrize("cin,cout,h,w,B", [(40, 64, 6, 10, 3), (8, 40, 4, 70, 2)])
def test_dense_weight_gradient_of_operands_that_are_not_finite(A, cin, cout, h, w, B):
    rng = np.random.default_rng(6)
    x = rng.standard_normal((B, cin, h, w)).astype(np.float32)
    dy = rng.standard_normal((B, cout, h, w)).astype(np.float32)
    x[0, 1, 2, w - 1] = np.inf       # (at the row's end: the next column is padding)
    x[1, 5, 0, 3] = np.nan
    x[1, 7, h - 1, 0] = 3.4e38       # rounds to infinity in bf16
    dy[0, 3, 1, 1] = -np.inf
    dy[:, :, h - 1, :2] *= 1e-6
    dy[1, :, h - 2, :2] *= 1e-6
    G, ref = weight_gradient(A, x, dy)
    with np.errstate(all="ignore"):
        want = ref.astype(np.float32)
    fin = np.isfinite(want)
    assert not fin.all() and fin.any()
    np.testing.assert_array_equal(G[~fin], want[~fin])
    assert np.isfinite(G[fin]).all()
    big = np.abs(want) > 1e6
    np.testing.assert_allclose(G[fin & ~big], want[fin & ~big], rtol=1e-5, atol=1e-4)
    np.testing.assert_allclose(G[fin & big], want[fin & big], rtol=1e-5)


# One pointwise convolution whose weight gradient has few, long ranges so that its stage fits the static workspace: every block
# shape that adds up in 64 bits, with loads of four and single words
@pytest.mark.parametrize("cin,cout,h,B,shape", [(512, 512, 56, 22, 1), (520, 512, 55, 24, 1), (1024, 96, 55, 60, 2),
                                                (1024, 90, 56, 60, 2), (2048, 32, 56, 85, 3), (2048, 31, 55, 90, 3)])
def test_pointwise_weight_gradient_of_few_ranges(A, cin, cout, h, B, shape):
    import ctypes
    import torch
    lib, out = ctypes.CDLL(A.lib_path()), (ctypes.c_int * 3)()
    parts = max(1, min(-(-768 // (-(-cin // 32) * -(-cout // 32))), B * h * h // 128))
    lib.ast_pw_wgrad_choice(B, cin, cout, h * h, parts, out)
    assert tuple(out) == (shape, parts, 1)
    st = A.Stage([conv(cin, cout, 1)], B, 1, 1, (cin, h, h), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    assert st.memory()[3] <= 32 << 20
    gen_ = torch.Generator(device="cuda")
    gen_.manual_seed(9)
    w = torch.randn(cout, cin, generator=gen_, device="cuda")
    st.set_params(w.cpu().numpy().ravel())
    x = torch.randn(B, cin, h, h, generator=gen_, device="cuda").clamp_(min=0)
    g = torch.randn(B, cout, h, h, generator=gen_, device="cuda")
    y, dx, dx2 = torch.empty_like(g), torch.empty_like(x), torch.empty_like(x)
    st.forward(0, x, None, y, None)
    st.backward(0, g, dx)
    G = st.get_grads()
    st.step(0.0, 0.0)
    st.forward(0, x, None, y, None)
    st.backward_static(0, g, dx2)
    np.testing.assert_array_equal(G, st.get_grads())
    assert torch.equal(dx, dx2)
    st.close()
    ref = torch.zeros(cout, cin, dtype=torch.float64, device="cuda")
    err = tot = 0.0
    for n in range(B):
        gn, xn = g[n].reshape(cout, -1).double(), x[n].reshape(cin, -1).double()
        ref += gn @ xn.t().contiguous()
        d = w.double().t().contiguous() @ gn
        err += float((dx[n].reshape(cin, -1).double() - d).pow(2).sum())
        tot += float(d.pow(2).sum())
    G = torch.from_numpy(G).cuda().reshape(cout, cin).double()
    assert float((G - ref).norm() / ref.norm()) <= BOUND_W
    assert (err / tot) ** 0.5 <= bound(cout)


@pytest.mark.parametrize("cin,cout,h,w,B,skip", [(8, 24, 1750, 1750, 2, False), (24, 8, 1747, 1749, 1, False), (33, 40, 1620, 1620, 1, True)])
def test_pointwise_planes_past_32_bit_offsets(A, cin, cout, h, w, B, skip):
    """... stay on the matrix cores (a wavefront addresses two samples from its first pixel on)."""
    import torch
    assert [pw_choice(d, B, cin, cout, h * w) for d in (0, 1)] == [FAR, FAR]
    layers = [conv(cin, cout, 1, bias=True)]
    if skip:   # the skip gradient is added by the input gradient's product
        layers = [simple("res_begin")] + layers + [conv(cout, cin, 1), simple("res_add")]
    st = A.Stage(layers, B, 1, 1, (cin, h, w), "f32", "nchw", True, stream=torch.cuda.current_stream().cuda_stream)
    gen_ = torch.Generator(device="cuda")
    gen_.manual_seed(2)
    r = lambda *s: torch.randn(*s, generator=gen_, device="cuda")
    p = r(st.num_params)
    st.set_params(p.cpu().numpy())
    x, g = r(B, cin, h, w), r(B, cin if skip else cout, h, w)
    y, dx = torch.empty_like(g), torch.empty_like(x)
    st.profile_begin("conv", 64)
    st.forward(0, x, None, y, None)
    st.backward(0, g, dx)
    names = set(st.profile_end())
    assert names == {"pw_conv_f32_far_kernel", "pw_wgrad_f32_kernel"} or names == {"pw_conv_f32_far_kernel"}, names
    G = torch.from_numpy(st.get_grads()).cuda().double()
    st.close()
    W, b = p[:cin * cout].view(cout, cin).double(), p[cin * cout:cin * cout + cout].double()
    V = p[cin * cout + cout:].view(cin, cout).double() if skip else None
    ref, e = torch.zeros_like(G), np.zeros(4)
    for n in range(B):
        xn, gn = x[n].view(cin, -1).double(), g[n].view(g.shape[1], -1).double()
        z = W @ xn + b[:, None]
        gz, yn = gn, z
        if skip:
            yn = V @ z + xn
            gz = V.t().contiguous() @ gn
            ref[cin * cout + cout:] += (gn @ z.t().contiguous()).ravel()
        dxn = W.t().contiguous() @ gz + (gn if skip else 0)
        ref[:cin * cout] += (gz @ xn.t().contiguous()).ravel()
        for i, (got, want) in enumerate(((y, yn), (dx, dxn))):
            e[2 * i] += float((got[n].view(want.shape).double() - want).pow(2).sum())
            e[2 * i + 1] += float(want.pow(2).sum())
    # (fp32 matrix instructions: a rounding per two terms, and two products behind each other)
    assert max(e[0] / e[1], e[2] / e[3]) ** 0.5 <= 1e-6
    G[cin * cout:cin * cout + cout] = 0   # (the bias gradient is another kernel's)
    assert float((G - ref).norm() / ref.norm()) <= 4e-7


@pytest.mark.parametrize("cin,mid,k", [(2048, 1024, 1), (512, 1024, 3)])
def test_time_of_the_packed_copies(A, cin, mid, k):
    """The update reads and writes 24 bytes a weight, the two split copies are 20: they take about as long."""
    import torch
    st = A.Stage([conv(cin, mid, k, 1, k // 2), conv(mid, cin, k, 1, k // 2)], 1, 1, 1, (cin, 4, 4), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    x = torch.randn(1, cin, 4, 4, device="cuda")
    y, dx, best = torch.empty_like(x), torch.empty_like(x), {}
    for _ in range(6):
        st.forward(0, x, None, y, None)
        st.backward(0, x, dx)
        st.profile_begin("", 64)
        st.step(0.0, 0.0)
        for name, (_, ms) in st.profile_end().items():
            best[name] = min(best.get(name, 1e9), ms)
    st.close()
    assert best["pw_pack_all_kernel"] <= 2.5 * best["sgd_kernel"], best


@pytest.mark.parametrize("sizes", [f[0] for f in FEWER_FORMS])
def test_dense_weight_gradient_of_few_partials(A, sizes):
    """A stage that has to fit the static workspace takes the staged fp32 kernel, which adds up in between."""
    import torch
    cin, cout, k, s, h, w, B = sizes
    out = wgrad_choice(B, cin, cout, h, w, k, s)
    st = A.Stage([conv(cin, cout, k, s, 1)], B, 1, 1, (cin, h, w), "f32", "nchw", True,
                 stream=torch.cuda.current_stream().cuda_stream)
    assert st.memory()[3] <= 32 << 20 < 36 * out[3] * cin * cout
    gen_ = torch.Generator(device="cuda")
    gen_.manual_seed(7)
    x, g = torch.randn(B, cin, h, w, generator=gen_, device="cuda"), torch.randn(B, cout, h, w, generator=gen_, device="cuda")
    y, dx = torch.empty_like(g), torch.empty_like(x)
    st.set_params(np.zeros(st.num_params, np.float32))
    st.forward(0, x, None, y, None)
    st.backward_static(0, g, dx)
    G = torch.from_numpy(st.get_grads()).cuda().view(cout, cin, 3, 3).double()
    st.close()
    xp, gm = torch.nn.functional.pad(x.double(), (1, 1, 1, 1)), g.double().permute(1, 0, 2, 3).reshape(cout, -1).contiguous()
    ref = torch.zeros_like(G)
    for u in range(3):
        for v in range(3):
            ref[:, :, u, v] = gm @ xp[:, :, u:u + h, v:v + w].permute(0, 2, 3, 1).reshape(-1, cin).contiguous()
    # (chains of at most 128 pixels of two terms each, test_tile_edges_gpu.py)
    assert float((G - ref).norm() / ref.norm()) <= 2.3e-7
