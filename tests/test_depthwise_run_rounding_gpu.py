"""Rounding of a BatchNorm, depthwise convolution, BatchNorm run in one launch per direction against 64 bits, where sums cancel:
no further off than the launches that it replaces."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

import harness
from asteroid_workloads.configs import bn, conv, simple
from test_parity_gpu import A  # noqa: F401  (the fixture)

C = 48


def in_64_bits(x, dy, p, k, s):
    q, xr, n = p.double().requires_grad_(), x.double().requires_grad_(), C * k * k
    g1, b1, w, g2, b2 = q.split([C, C, n, C, C])
    h = F.silu(F.batch_norm(xr, None, None, g1, b1, True, 0, 1e-5))
    h = F.conv2d(h, w.view(C, 1, k, k), None, s, k // 2, 1, C)
    y = F.silu(F.batch_norm(h, None, None, g2, b2, True, 0, 1e-5))
    y.backward(dy.double())
    return [y.detach(), xr.grad] + list(q.grad.split([C, C, n, C, C]))


# Values around `mean`: at 30 the variance is a small difference of the sums of squares.  Some errors are those of one rounding in
# each of 48 channels (of a mean, of an inverse deviation): they differ by a quarter between orders of addition, and half is
# allowed.  The mean of a BatchNorm's gradient taken off a rounded product makes its neighbour's gamma and beta 2 to 10 times as
# far off.
@pytest.mark.gpu
@pytest.mark.parametrize("mean", [0, 30])
@pytest.mark.parametrize("k,s,hw,B", [(3, 1, 28, 36), (5, 1, 30, 32), (3, 2, 56, 9), (5, 2, 31, 20), (3, 1, 14, 8)])
def test_no_further_off_than_separate_launches(A, monkeypatch, k, s, hw, B, mean):
    g = torch.Generator().manual_seed(3)
    ho, n = (hw - 1) // s + 1, C * k * k
    x, dy = torch.randn(B, C, hw, hw, generator=g) + mean, torch.randn(B, C, ho, ho, generator=g)
    one, zero = torch.ones(C), torch.zeros(C)
    p = torch.cat([one, zero, torch.randn(n, generator=g) / k + 0.5, one, zero])
    want = in_64_bits(x, dy, p, k, s)
    layers = [bn(C), simple("swish"), conv(C, C, k, s, k // 2, groups=C), bn(C), simple("swish")]
    errors = []
    for fuse in ("31", "15"):
        monkeypatch.setenv("ASTEROID_BN_FUSE", fuse)
        st = A.Stage(layers, B, 1, 1, (C, hw, hw), "f32", "nchw", True, stream=torch.cuda.current_stream().cuda_stream)
        st.set_params(p.numpy())
        xd, gd = x.cuda(), dy.cuda()
        y, dx = torch.empty_like(gd), torch.empty_like(xd)
        st.forward(0, xd, None, y)
        st.backward(0, gd, dx)
        torch.cuda.synchronize()
        G = torch.from_numpy(st.get_grads().copy())
        st.close()
        have = [y.cpu(), dx.cpu()] + list(G.split([C, C, n, C, C]))
        errors.append([harness.rel_l2(a, b) for a, b in zip(have, want)])
    assert (np.array(errors[0]) <= 1.5 * np.array(errors[1])).all(), errors
