"""BatchNorm, activation, depthwise convolution, BatchNorm, activation as one launch per direction: every form of its blocks
(strip of a thread, threads, values per thread) at planes that leave remainders, and the launches that take the same run apart,
against the oracle."""
import ctypes

import numpy as np
import pytest

import harness
import paper_2408_08015_amd as lib
from asteroid_workloads import gen
from asteroid_workloads.configs import bn, conv, simple
from test_parity_gpu import A, one  # noqa: F401  (A: the fixture)

SWISH, RELU6 = 4, 2


def choice(bwd, k, B, c, h, w, s, act):
    out = (ctypes.c_int * 3)()
    return tuple(out) if ctypes.CDLL(lib.lib_path()).ast_dws_choice(bwd, k, B, c, h, w, s, act, out) else None


# (kernel, stride, channels, h, w, B), the forward's and the backward's form
FORMS = [
    ((3, 1, 5, 7, 7, 3), (1, 256, 4), (1, 256, 4)),
    ((3, 1, 3, 1, 1, 5), (1, 256, 4), (1, 256, 4)),         # planes of one pixel
    ((3, 1, 4, 9, 16, 4), (4, 256, 4), (4, 256, 4)),        # bands of one row
    ((3, 1, 4, 6, 10, 27), (2, 512, 4), (2, 512, 4)),
    ((3, 1, 3, 27, 27, 4), (1, 512, 8), (1, 512, 8)),       # a last band of fewer rows
    ((3, 1, 3, 14, 14, 31), (2, 1024, 8), (2, 1024, 8)),
    ((3, 1, 2, 27, 29, 13), (1, 1024, 16), (1, 1024, 16)),
    ((3, 1, 2, 31, 31, 32), (1, 1024, 32), (1, 1024, 32)),
    ((3, 1, 2, 28, 30, 34), (2, 1024, 32), (2, 1024, 32)),
    ((3, 1, 2, 28, 28, 32), (4, 1024, 32), (4, 1024, 32)),
    ((3, 2, 4, 7, 9, 5), (1, 256, 4), (1, 256, 4)),         # odd planes: the last quads reach past them
    ((3, 2, 4, 14, 14, 8), (1, 512, 4), (1, 256, 4)),
    ((3, 2, 3, 28, 28, 8), (2, 1024, 8), (2, 512, 4)),
    ((3, 2, 2, 56, 56, 8), (4, 1024, 32), (4, 1024, 8)),
    ((3, 2, 2, 47, 45, 9), (1, 1024, 32), (1, 1024, 8)),
    ((5, 1, 5, 5, 3, 4), (1, 256, 4), (1, 256, 4)),
    ((5, 1, 3, 15, 15, 8), (1, 512, 4), (1, 512, 4)),
    ((5, 1, 2, 12, 20, 30), (4, 1024, 8), (4, 1024, 8)),
    ((5, 1, 2, 30, 30, 32), (2, 1024, 32), (2, 1024, 32)),
    ((5, 2, 4, 15, 15, 8), (1, 512, 4), (1, 256, 4)),
    ((5, 2, 2, 60, 60, 8), (2, 1024, 32), (2, 1024, 8)),
    ((5, 2, 2, 24, 32, 40), (4, 1024, 32), (4, 1024, 8)),
    ((3, 2, 4, 7, 28, 8), (1, 512, 4), (1, 256, 4)),        # an odd number of rows of an even number of columns: single ones,
    ((5, 2, 3, 5, 24, 6), (1, 256, 4), (1, 256, 4)),        # as the quads of the last row reach past it
    ((3, 2, 2, 47, 56, 9), (1, 1024, 32), (1, 1024, 8)),
    ((3, 2, 3, 28, 8, 9), (4, 512, 4), (4, 256, 4)),
    ((3, 1, 3, 9, 28, 11), (4, 512, 8), (4, 512, 8)),
    ((3, 1, 2, 45, 45, 16), None, None),                    # no thread for every strip
    ((3, 1, 2, 56, 56, 11), None, None),                    # a channel larger than a block
]


@pytest.mark.parametrize("sizes,forward,backward", FORMS)
def test_form(sizes, forward, backward):
    k, s, c, h, w, B = sizes
    act = SWISH if k == 5 else RELU6
    assert choice(0, k, B, c, h, w, s, act) == forward
    assert choice(1, k, B, c, h, w, s, act) == backward


def test_forms_that_stay_apart():
    assert choice(0, 3, 4, 8, 14, 14, 1, 0) is None and choice(0, 5, 4, 8, 14, 14, 1, RELU6) is None


# Blocks of 32 values a thread: one launch where their channels fill rounds of 256 well enough, on either side of that line
@pytest.mark.parametrize("sizes,taken", [
    ((5, 1, 8, 31, 31, 27), False), ((5, 1, 64, 31, 31, 27), False), ((5, 1, 240, 31, 31, 27), True), ((5, 1, 272, 31, 31, 27), False),
    ((5, 1, 8, 28, 28, 32), False), ((5, 1, 96, 28, 28, 32), True), ((3, 1, 8, 31, 31, 27), False), ((3, 1, 96, 31, 31, 27), True),
    ((3, 1, 8, 28, 28, 32), True), ((5, 2, 8, 30, 30, 32), False), ((5, 2, 240, 30, 30, 32), True), ((5, 2, 8, 56, 56, 9), True),
    ((5, 1, 8, 14, 14, 64), True), ((3, 1, 8, 7, 7, 64), True),          # 16 values and fewer: always
])
def test_one_launch_where_it_is_faster(monkeypatch, sizes, taken):
    k, s, c, h, w, B = sizes
    act = "swish" if k == 5 else "relu6"
    layers = [bn(c), simple(act), conv(c, c, k, s, k // 2, groups=c), bn(c), simple(act)]

    def workspace():   # (a run in one launch has no partials in it)
        return lib.plan_memory(layers, B, 1, 1, (c, h, w), "f32", "nchw", True)[3]

    monkeypatch.delenv("ASTEROID_BN_FUSE", raising=False)
    got = workspace()
    monkeypatch.setenv("ASTEROID_BN_FUSE", "31" if taken else "15")
    assert got == workspace()
    monkeypatch.setenv("ASTEROID_BN_FUSE", "15" if taken else "31")
    assert got != workspace()


# fuse: the bit mask of ASTEROID_BN_FUSE; without 16 the run is taken apart, with it it is one launch wherever a channel fits
@pytest.mark.gpu
@pytest.mark.parametrize("fuse", [31, 15])
@pytest.mark.parametrize("grad", [True, False])
@pytest.mark.parametrize("sizes", [f[0] for f in FORMS])
def test_run(A, monkeypatch, sizes, grad, fuse):
    k, s, c, h, w, B = sizes
    if fuse == 15 and not grad:
        pytest.skip("the launches that take the run apart are the same ones")
    monkeypatch.setenv("ASTEROID_BN_FUSE", str(fuse))
    acts = ("swish", "swish") if k == 5 else ("relu", "relu6") if c % 2 else ("relu6", "relu")
    layers = [bn(c), simple(acts[0]), conv(c, c, k, s, k // 2, groups=c), bn(c), simple(acts[1])]
    # an element whose value in front of an activation is within its fp32 rounding of an edge may take the other slope, and its
    # whole gradient differs then: the first inputs without one (the rounding of values up to 6: 1e-6)
    for seed in range(40):
        cfg = one(layers, (c, h, w), B=B, M=2, seed=seed)
        cfg.needs_input_grad = grad
        inp = gen.make_inputs(cfg, randomize_affine=True)
        ora, st = harness.run_oracle(cfg, inp, rounds=1, keep_acts=True)
        edge = min(np.abs(st.acts[m][layer] - v).min() for m in range(2) for layer in (0, 3) for v in (0, 6))
        if k == 5 or edge > 4e-6:
            break
    else:
        pytest.fail("no inputs away from the edges")
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    # sums of at most 32768 terms in chains of 32 additions and 64-bit ones, as exact as their terms (1e-7 each), and the
    # differences of a BatchNorm's backward, which lose a digit or two
    assert sc["r0.y"] <= 2e-6
    if grad:
        assert sc["r0.dx"] <= 1e-5
    for name, err in sc["r0.G_all"]:
        assert err <= 1e-4, (name, err)


# the activation in front of the convolution is formed inside the launch; asked for, it is formed again (with ReLU and ReLU6 it
# cannot be asked for, as where the run is taken apart)
@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [f[0] for f in FORMS if f[0][:2] != (3, 2) and f[1]][::4])
def test_activation_in_front(A, sizes):
    k, s, c, h, w, B = sizes
    for act in ("swish", "relu6") if k == 3 else ("swish",):
        layers = [bn(c), simple(act), conv(c, c, k, s, k // 2, groups=c), bn(c), simple(act)]
        cfg = one(layers, (c, h, w), B=B, M=1)
        inp = gen.make_inputs(cfg, randomize_affine=True)
        _, st = harness.run_oracle(cfg, inp, rounds=1, keep_acts=True)
        _, dbg, _ = harness.run_hip(cfg, inp, rounds=1, debug_layers=[0, 1])
        assert list(dbg) == ([1] if act == "swish" else [])
        if dbg:   # (a BatchNorm in fp32 from statistics in 64 bits)
            assert harness.rel_l2(dbg[1], st.acts[0][1]) <= 5e-7
