"""Weight gradients of a stage's linear layers in one launch: products formed whole, in shares of their rows, and in shares of two
counts, against the oracle; and a stage that the partials of the shares would take past the static workspace."""
import ctypes

import numpy as np
import pytest

import harness
import paper_2408_08015_amd as lib
from asteroid_workloads import gen
from asteroid_workloads.configs import encoder_layer, linear
from test_parity_gpu import A, one_bf16  # noqa: F401  (A: the fixture)


def shares(rows, sizes):
    n = len(sizes)
    cin, cout, out = ((ctypes.c_int * n)(*v) for v in ([s[0] for s in sizes], [s[1] for s in sizes], [0] * n))
    ctypes.CDLL(lib.lib_path()).ast_wgrad_shares(ctypes.c_long(rows), n, cin, cout, out)
    return list(out)


def products(d, ffn, layers):
    """In the order of the backward pass."""
    return [(ffn, d), (d, ffn), (d, d), (d, 3 * d)] * layers


@pytest.mark.parametrize("rows,sizes,want", [
    (4096, products(512, 2048, 6), {1, 8}),       # 288 tiles on 256 compute units
    (10240, products(768, 3072, 4), {1, 2, 4}),
    (864, products(768, 3072, 2), {1}),           # 216 tiles: one round of whole ones
    (2560, products(256, 1024, 1), {11}),         # twelve tiles
    (47, products(256, 1024, 1), {1}),
    (192, products(256, 1024, 1), {1}),           # two shares would be shorter than four steps
])
def test_shares(rows, sizes, want):
    got = shares(rows, sizes)
    assert set(got) == want
    assert all(s == 1 or -(-rows // (-(-(-(-rows // s)) // 48) * 48)) == s for s in got)   # no share is empty


# d, heads, ffn, layers, S, B: rows that are no multiple of a share or of 48, features that fill no tile
@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,ffn,layers,S,B", [(256, 4, 1024, 1, 128, 17), (192, 3, 776, 1, 96, 13), (128, 2, 264, 2, 64, 9)])
def test_encoder(A, d, heads, ffn, layers, S, B):
    assert max(shares(B * S, products(d, ffn, layers))) > 1
    cfg = one_bf16(encoder_layer(d, heads, ffn) * layers, (S, d), "bsd", B=B, M=1)
    inp = gen.make_inputs(cfg, randomize_affine=True)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    sc = harness.score(cfg, hip, ora)
    assert max(sc["r0.y"], sc["r0.dx"]) <= 2e-2
    for name, err in sc["r0.G_all"]:
        assert err <= 2e-2, (name, err)


@pytest.mark.gpu
def test_stage_at_the_static_workspace(A):
    # 1408 rows: five shares are 40 MB of partials, the stage without them 31.5
    d, ffn, S, B = 512, 1024, 128, 11
    assert min(shares(B * S, products(d, ffn, 1))) > 2
    assert lib.plan_memory(encoder_layer(d, 8, ffn), B, 1, 1, (S, d), "bf16", "bsd", True)[3] <= 32 << 20
    cfg = one_bf16(encoder_layer(d, 8, ffn), (S, d), "bsd", B=B, M=1)
    inp = gen.make_inputs(cfg)
    a, _, _ = harness.run_hip(cfg, inp, rounds=1)
    b, _, _ = harness.run_hip(cfg, inp, rounds=1, static_backward=True)
    assert (a[0]["G"] == b[0]["G"]).all() and (a[0]["dx"] == b[0]["dx"]).all()


# a layer between two whose operands lie in the caller's buffers (those have launches of their own)
@pytest.mark.gpu
def test_layers_at_the_ends_of_a_stage(A):
    cfg = one_bf16([linear(256, 520), linear(520, 264), linear(264, 128)], (96, 256), "bsd", B=30, M=2)
    inp = gen.make_inputs(cfg)
    ora, _ = harness.run_oracle(cfg, inp, rounds=1)
    hip, _, _ = harness.run_hip(cfg, inp, rounds=1)
    for name, err in harness.score(cfg, hip, ora)["r0.G_all"]:
        assert err <= 1e-2, (name, err)


# more sums than the reduction's table holds: nothing adds up partials there, and the product behind it is formed whole
@pytest.mark.gpu
def test_stage_longer_than_the_reduction_table(A, monkeypatch):
    import torch
    d, S, B, n = 64, 16, 24, 32768   # two sums to a normalisation, 65535 in the table
    assert shares(B * S, [(d, d)]) == [2]
    ln = dict(kind="layernorm", d=d, eps=1e-5)
    layers = [ln] * (n - 1) + [linear(d, d), ln]
    g = torch.Generator().manual_seed(3)
    x, dy = (torch.randn(B, S, d, generator=g).bfloat16().cuda() for _ in range(2))
    got = []
    for group in ("1", "0"):
        monkeypatch.setenv("ASTEROID_WGRAD_GROUP", group)
        st = A.Stage(layers, B, 1, 1, (S, d), "bf16", "bsd", stream=torch.cuda.current_stream().cuda_stream)
        p = np.tile(np.repeat(np.float32([1, 0]), d), n)
        at = 2 * d * (n - 1)
        w = torch.randn(d * d + d, generator=torch.Generator().manual_seed(4)).mul(0.1).numpy()
        st.set_params(np.concatenate([p[:at], w, p[:2 * d]]))
        y, dx = torch.empty_like(dy), torch.empty_like(x)
        st.forward(0, x, None, y)
        st.backward(0, dy, dx)
        torch.cuda.synchronize()
        got.append(st.get_grads()[at:at + d * d + d])
        st.close()
    # the same products in another order of fp32 additions: 384 of them
    assert np.linalg.norm(got[1]) > 0 and harness.rel_l2(got[0], got[1]) < 1e-5
