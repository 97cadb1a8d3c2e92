"""fp32 products on the bf16 matrix cores with their operands split in three: the kernel forms at sizes on either side of
their rules, their rounding error, and operands that are not finite."""
import numpy as np
import pytest

import harness
from asteroid_workloads import gen
from asteroid_workloads.configs import conv, simple
from test_parity_gpu import A, one  # noqa: F401  (A: the fixture)

pytestmark = pytest.mark.gpu

# Relative error of a product of normal matrices: about 2^-25 from the last rounding plus a random walk of one rounding per
# 16 terms, 6e-8 + 2^-25 * sqrt(K / 16) / 2; the fp32 matrix instructions, which round every second term, are at
# 2^-25 * sqrt(K / 2) and more.  Weight gradients: chains of at most 32 roundings, 1e-7 measured.
BOUND_W = 2e-7


def bound(k):
    return 1.2e-7 + 2.0 ** -24 * (k / 16) ** 0.5


@pytest.mark.parametrize("cin,cout,h,w,B", [
    (15, 33, 5, 7, 3),        # one group of 16 channels, odd planes, a second row tile of one row
    (17, 31, 9, 9, 2),
    (96, 576, 14, 14, 1),     # K split over four wavefronts, forward and back; few pixels
    (576, 96, 7, 7, 2),       # ... over eight
    (528, 264, 7, 7, 10),     # ... four with two row tiles, the last pair has one
    (81, 40, 25, 24, 32),     # two pixels per lane: 600 per plane
    (80, 72, 24, 24, 90),     # ... and two row tiles; three of them one by one
    (80, 72, 25, 25, 20),     # odd planes: one pixel per lane, two row tiles
    (16, 104, 56, 56, 20),    # short contractions: all row tiles in one wavefront
    (33, 264, 28, 28, 36),    # ... nine tiles in two shares
    (64, 96, 56, 56, 24),
    (40, 40, 1, 3, 70),       # planes of three pixels: a wavefront spans a dozen samples
])
def test_pointwise_forms(A, cin, cout, h, w, B):
    cfg = one([conv(cin, cout, 1)], (cin, h, w), B=B, M=1)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    assert sc["r0.y"] <= bound(cin)
    assert sc["r0.dx"] <= bound(cout)
    assert harness.rel_l2(hip[0]["G"], ora[0]["G"]) <= BOUND_W


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


@pytest.mark.parametrize("cin,cout,h,B", [(24, 40, 6, 3), (160, 40, 7, 2), (72, 72, 24, 90), (24, 104, 56, 20)])
def test_pointwise_operands_that_are_not_finite(A, cin, cout, h, B):
    """An infinity or NaN reaches the outputs that its definition gives and no others, with the right sign, and the largest
    finite values are still values."""
    import torch
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
