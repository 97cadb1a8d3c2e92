"""Short passes that ride with their neighbours: a ReLU or ReLU6 that stands alone at a residual block's end with the
BatchNorm or the addition in front, and the sum of a few rows' losses with their softmax."""
import numpy as np
import pytest

import harness
from asteroid_workloads import gen
from asteroid_workloads.configs import bn, conv, linear, simple
from test_parity_gpu import A, one  # noqa: F401  (A: the fixture)

pytestmark = pytest.mark.gpu


def layers_of(two, act, c, mid):
    main = [conv(c, mid, 1), bn(mid), simple("relu"), conv(mid, c, 1), bn(c)]
    if two:
        return [simple("res_begin")] + main + [simple("res_swap"), conv(c, c, 1), bn(c), simple("res_add"), simple(act)]
    return [simple("res_begin")] + main + [simple("res_add"), simple(act)]


# planes of whole vectors and odd ones, in one launch per BatchNorm (at most 8192 elements per channel) and in two; the last two:
# tensors of an odd number of elements, where behind an addition the activation keeps a pass of its own forward
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("act,c,mid,hw,B", [("relu", 16, 24, 8, 3), ("relu6", 24, 16, 7, 3), ("relu", 16, 16, 56, 4),
                                            ("relu6", 16, 24, 45, 6), ("relu", 5, 7, 7, 3), ("relu6", 5, 7, 45, 5)])
def test_activation_behind_a_residual_block(A, two, act, c, mid, hw, B):
    # one block in front of another: the first one's activation lies in the stash, the second one's is the stage's output
    layers = layers_of(two, act, c, mid) + layers_of(False, act, c, mid)
    cfg = one(layers, (c, hw, hw), B=B, M=1)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    assert sc["r0.y"] <= 2e-6
    # (an element within the rounding of an activation's edge takes another slope: its whole gradient differs)
    assert sc["r0.dx"] <= 1e-3
    # the statistics pass of the backward forms the masked gradient and leaves gamma's and beta's: every parameter gradient
    # stands on it
    for name, err in sc["r0.G_all"]:
        assert err <= 1e-3, (name, err)


# the sum in front of that activation is written only where something else reads it; asked for, it is formed again
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("act,hw,B", [("relu", 8, 3), ("relu6", 7, 3), ("relu", 56, 4)])
def test_sum_in_front_of_that_activation(A, two, act, hw, B):
    layers = layers_of(two, act, 16, 24) + layers_of(False, act, 16, 24)
    at = len(layers_of(two, act, 16, 24)) - 2   # the addition; the activation behind it
    cfg = one(layers, (16, hw, hw), B=B, M=1)
    inp = gen.make_inputs(cfg)
    _, dbg, _ = harness.run_hip(cfg, inp, rounds=1, debug_layers=[at, at + 1])
    pre, post = dbg[at], dbg[at + 1]
    assert pre.min() < 0
    want = np.clip(pre, 0, 6 if act == "relu6" else None)
    # (one rounding of a fused multiply-add and one of the addition)
    np.testing.assert_allclose(post, want, rtol=2.4e-7, atol=2.4e-7 * np.abs(pre).max())


# on either side of sixteen rows and 64 classes, the largest heads that one block takes
@pytest.mark.parametrize("B,classes", [(1, 2), (4, 10), (16, 64), (17, 64), (16, 65)])
def test_loss_of_few_rows(A, B, classes):
    cfg = one([simple("global_avgpool"), linear(24, classes), simple("softmax_ce")], (24, 5, 5), B=B, M=2)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    # (a few roundings each: the exponential, the sum of at most 65 of them, the logarithm)
    assert max(sc["r0.y"], sc["r0.dx"], sc["r0.loss"]) <= 2e-6
