"""The weight gradient of a bf16 3x3 convolution with all taps in a wavefront, and the rule that takes it."""
import ctypes

import numpy as np
import pytest

import harness  # noqa: F401
import paper_2408_08015_amd as lib
from asteroid_workloads.configs import conv
from test_parity_gpu import A  # noqa: F401  (the fixture)


def partials(B, h, w, cin, cout):
    return ctypes.CDLL(lib.lib_path()).ast_conv_wgrad_taps_choice(B, h, w, cin, cout)


# cin, cout, h, w, B: partials
SIZES = [
    ((8, 8, 1, 1, 1), 1),              # one pixel
    ((8, 24, 5, 5, 1), 1),             # less than a chunk of pixels
    ((16, 40, 15, 15, 1), 1),          # a chunk exactly
    ((40, 64, 15, 31, 1), 2),          # two
    ((200, 72, 9, 7, 23), 8),          # channels that fill no tile in either operand
    ((64, 64, 1, 50, 33), 14),         # images of one row, of one column
    ((64, 64, 50, 1, 33), 14),
    ((32, 32, 2, 300, 3), 11),         # rows longer than a chunk
    ((96, 96, 45, 45, 6), 50),
    ((16, 32, 56, 56, 24), 305),       # one tile: as many ranges as blocks that run together
    ((256, 256, 45, 45, 10), 8),       # 64 tiles
]


@pytest.mark.parametrize("sizes,want", SIZES)
def test_choice(sizes, want):
    cin, cout, h, w, B = sizes
    assert partials(B, h, w, cin, cout) == want


def test_choice_of_the_tiles_of_256_channels():
    assert partials(10, 45, 45, 256, 256) and not partials(32, 56, 56, 256, 256)   # many tiles, many pixels
    assert not partials(1, 3, 1200, 64, 64)                                        # rows that do not fit a block's LDS


def test_partials_that_would_not_fit_the_static_workspace(monkeypatch):
    """A stage that the partials for speed would take past it has no more of them than other kernels leave."""
    layers = [conv(32, 96, 3, 1, 1, bias=True), conv(96, 32, 3, 1, 1, bias=True)] * 2

    def workspace():
        return lib.plan_memory(layers, 10, 1, 1, (32, 45, 45), "bf16", "nhwc", True)[3]

    got, more = workspace(), partials(10, 45, 45, 32, 96)
    monkeypatch.setenv("ASTEROID_CONV_WGRAD", "0")
    assert got <= workspace() <= 32 << 20 < workspace() + 4 * (more - 28) * 9 * 32 * 96 * 4


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [s[0] for s in SIZES])
def test_whole_numbers(A, monkeypatch, sizes):
    """Whole numbers of at most 2 in either operand: every sum is below 2^24, so that the gradients are those of integers."""
    import torch
    cin, cout, h, w, B = sizes
    assert B * h * w * 4 < 1 << 24
    dev, g = torch.device("cuda:0"), torch.Generator().manual_seed(5)
    x, dy = (torch.randint(-2, 3, (B, h, w, c), generator=g) for c in (cin, cout))
    got = []
    for taps in ("1", "0"):
        monkeypatch.setenv("ASTEROID_CONV_WGRAD", taps)
        st = A.Stage([conv(cin, cout, 3, 1, 1, bias=True)], B, 1, 1, (cin, h, w), "bf16", "nhwc")
        st.set_params(np.zeros(st.num_params, np.float32))
        xd, gd = x.to(dev, torch.bfloat16), dy.to(dev, torch.bfloat16)
        y, dx = torch.empty_like(gd), torch.empty_like(xd)
        torch.cuda.synchronize()
        st.forward(0, xd, None, y)
        st.backward(0, gd, dx)
        got.append(st.get_grads())
        st.close()
    xp = torch.nn.functional.pad(x.float(), (0, 0, 1, 1, 1, 1))
    rows = dy.float().reshape(-1, cout).t()
    want = torch.stack([rows @ xp[:, u:u + h, v:v + w].reshape(-1, cin) for u in range(3) for v in range(3)])  # [tap][cout][cin]
    want = np.concatenate([want.permute(1, 2, 0).reshape(-1).numpy(), dy.sum((0, 1, 2)).float().numpy()])
    for have in got:
        assert np.array_equal(have, want)


@pytest.mark.gpu
@pytest.mark.parametrize("of", ["x", "dy"])
@pytest.mark.parametrize("sizes", [(24, 40, 9, 7, 3), (64, 64, 1, 50, 33), (64, 64, 50, 1, 33), (40, 64, 15, 31, 8), (32, 32, 2, 300, 3)])
def test_values_that_are_not_finite(A, sizes, of):
    """An infinity or a NaN reaches the weights whose products it is part of, and no others: pixels in the corners and at the
    edges of images, and at the ends of what a block works on."""
    import torch
    cin, cout, h, w, B = sizes
    assert partials(B, h, w, cin, cout)
    g = torch.Generator().manual_seed(5)
    x, dy = (torch.randint(1, 3, (B, h, w, c), generator=g).float() for c in (cin, cout))
    t, n = (x, cin) if of == "x" else (dy, cout)
    t = t.view(B * h * w, n)
    at = [0, w - 1, (h - 1) * w, h * w - 1, B * h * w - 1]
    for q in range(255, B * (h + 1) * (w + 1), 256):   # on either side of every 256th pixel of the order that the kernel walks
        row, col = divmod(q, w + 1)
        img, r = divmod(row, h + 1)
        at.append((img * h + min(r, h - 1)) * w + min(col, w - 1))
    for i, p in enumerate(at):   # (each in a channel of its own, as far as there are)
        t[min(p + i % 2, B * h * w - 1), (3 * i) % n] = float("nan") if i % 4 == 2 else float("inf")
    dev = torch.device("cuda:0")
    st = A.Stage([conv(cin, cout, 3, 1, 1)], B, 1, 1, (cin, h, w), "bf16", "nhwc")
    st.set_params(np.zeros(st.num_params, np.float32))
    xd, gd = x.to(dev, torch.bfloat16), dy.to(dev, torch.bfloat16)
    y, dx = torch.empty_like(gd), torch.empty_like(xd)
    torch.cuda.synchronize()
    st.forward(0, xd, None, y)
    st.backward(0, gd, dx)
    have = st.get_grads().reshape(cout, cin, 3, 3)
    st.close()
    want = np.zeros((cout, cin, 3, 3), np.float32)
    for u in range(3):
        for v in range(3):   # the pairs of pixels that there are
            a = x[:, max(u - 1, 0):h + min(u - 1, 0), max(v - 1, 0):w + min(v - 1, 0)].reshape(-1, cin)
            b = dy[:, max(1 - u, 0):h + min(1 - u, 0), max(1 - v, 0):w + min(1 - v, 0)].reshape(-1, cout)
            want[:, :, u, v] = (b.t() @ a).numpy()
    assert 0 < np.isfinite(want).sum() < want.size
    assert np.array_equal(have, want, equal_nan=True)
