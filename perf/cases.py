"""The rounds of a pipeline stage that are timed, and how.

One pass is one HPP-Round as a training program makes it: M micro-batches through forward and backward in
one-forward-one-backward order behind K warm-up forwards, the momentum-SGD update, and the read-back of the
optimizer's velocity into a pinned host buffer (the part of a checkpoint that holds the accumulated gradient).
The stages are those of asteroid_workloads.configs, at their stated sizes and at others of the same kind.

A case:
  family   which layer list (see _config)
  B, M     samples per micro-batch, micro-batches per round
  K        activation stashes (warm-up forwards); 1 unless a later stage is waited for
  fwd      the forward passes run on a second stream (asteroid_stage_set_forward_stream)
  static   the backward passes go through asteroid_stage_backward_static
and the sizes that the family takes.
"""
import ctypes
import math

import torch

import paper_2408_08015_amd as asteroid
from asteroid_workloads import configs, gen

LR, MOMENTUM = 1e-5, 0.9   # a warm-up rate

BRANCH_SCALE = 0.2


def _case(family, B, M, K=1, fwd=False, static=False, **sizes):
    return dict(family=family, B=B, M=M, K=K, fwd=fwd, static=static, **sizes)


def listed():
    return [
        # The profiler's smallest call: one inverted-residual block, one sample, one micro-batch.  Nothing but
        # launch latency.
        dict(_case("block", 1, 1, cin=96, cout=96, stride=1, hw=14), name="block_one_sample"),
        # A whole small network with its loss on one device: still bound by launches.
        dict(_case("tiny", 4, 2, hw=16), name="tiny_cnn"),
        # The fp32 stage of the benchmark: MobileNetV2 blocks at 56x56, ordinary micro-batches.
        dict(_case("mbv2", 32, 4, hw=56), name="mbv2_stage"),
        # The same stage as an early member of a pipeline: three stashes, forwards on a stream of their own, the
        # uneven share of a micro-batch that the planner gives a slower device, planes of odd width.
        dict(_case("mbv2", 13, 5, K=3, fwd=True, hw=54), name="mbv2_stage_odd_share"),
        # A whole model on one device: many short dependent launches on shrinking planes.
        dict(_case("mbv2_full", 8, 8, hw=224), name="mbv2_full"),
        # The headline of the benchmark: three bf16 3x3 convolutions, large matrix products.
        dict(_case("vgg", 32, 4, hw=56, cin=128, c=256), name="vgg_stage"),
        # bf16 convolutions whose channels and pixels fill no tile.
        dict(_case("vgg", 6, 4, hw=45, cin=48, c=96), name="vgg_ragged"),
        # The transformer stage of the benchmark.
        dict(_case("bert", 32, 4, S=128, d=512, heads=8, ffn=2048, nlayers=6), name="bert_stage"),
        # A wider, shorter transformer stage early in a pipeline: 864 rows fill no tile.
        dict(_case("bert", 9, 4, K=3, fwd=True, S=96, d=768, heads=12, ffn=3072, nlayers=2), name="bert_stage_wide"),
        # EfficientNet-B1 blocks: 5x5 depthwise, swish, squeeze-and-excitation.
        dict(_case("effnet", 32, 4, hw=60), name="effnet_stage"),
        # ResNet50's first block group: dense fp32 3x3 convolutions, projection shortcut, the widest tensors.
        dict(_case("resnet", 32, 4, hw=56), name="resnet_stage"),
        # The largest: the whole ResNet50 on one device.
        dict(_case("resnet_full", 8, 8, hw=224), name="resnet_full"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["block", "block", "tiny", "mbv2", "mbv2", "mbv2_full", "vgg", "vgg", "bert", "bert",
                         "effnet", "resnet", "effnet_full", "resnet_full"])
    M = rng.randint(1, 6)
    deep = rng.random() < 0.3 and M >= 2   # an early stage of a pipeline
    K = min(M, rng.choice([2, 3])) if deep else 1
    fwd = deep and rng.random() < 0.7
    if family == "block":   # the units of the whole models, as the profiler times them
        stride = rng.choice([1, 1, 1, 2])
        cin, hw = rng.choice([(16, 112), (24, 56), (32, 28), (64, 14), (96, 14), (160, 7)])
        cout = cin if stride == 1 else rng.choice([24, 32, 64, 160])
        return _case("block", _log_int(rng, 1, 64), 1, static=rng.random() < 0.2 and hw <= 14, cin=cin, cout=cout,
                     stride=stride, hw=hw)
    if family == "tiny":
        return _case("tiny", _log_int(rng, 1, 24), M, K, fwd, static=rng.random() < 0.2, hw=rng.randint(8, 28))
    if family == "mbv2":
        return _case("mbv2", _log_int(rng, 3, 40), M, K, fwd, hw=rng.randint(20, 64))
    if family == "mbv2_full":
        return _case("mbv2_full", _log_int(rng, 2, 16), M, K, fwd, hw=rng.choice([128, 160, 192, 224]))
    if family == "vgg":
        if rng.random() < 0.5:
            cin, c = rng.choice([64, 128, 192, 256]), rng.choice([64, 128, 192, 256])
        else:
            cin, c = 8 * rng.randint(2, 20), 8 * rng.randint(4, 28)
        return _case("vgg", _log_int(rng, 2, 40), M, K, fwd, hw=rng.randint(14, 60), cin=cin, c=c)
    if family == "bert":
        heads = rng.choice([4, 6, 8, 12])
        return _case("bert", _log_int(rng, 1, 40), M, K, fwd, S=32 * rng.randint(1, 8), d=64 * heads, heads=heads,
                     ffn=256 * heads, nlayers=rng.randint(1, 4))
    if family == "effnet":
        return _case("effnet", _log_int(rng, 3, 40), M, K, fwd, hw=rng.randint(24, 64))
    if family == "resnet":
        return _case("resnet", _log_int(rng, 2, 32), M, K, fwd, hw=rng.randint(14, 56))
    if family == "effnet_full":
        return _case("effnet_full", _log_int(rng, 1, 8), M, K, fwd, hw=rng.choice([128, 160, 192, 224, 240]))
    return _case("resnet_full", _log_int(rng, 2, 8), M, K, fwd, hw=rng.choice([128, 160, 192, 224]))


def _config(case):
    B, M = case["B"], case["M"]
    if case["family"] == "block":
        hw, cin = case["hw"], case["cin"]
        return configs.StageConfig("block", configs.irb(cin, case["cout"], case["stride"], 6), B, M, (cin, hw, hw),
                                   "f32", "nchw", True, 0)
    make = {"tiny": configs.cfg1, "mbv2": configs.cfg2, "mbv2_full": configs.cfg3, "vgg": configs.cfg4,
            "bert": configs.cfg5, "effnet": configs.cfg6, "resnet": configs.cfg7, "effnet_full": configs.effnetb1,
            "resnet_full": configs.resnet50}[case["family"]]
    sizes = {k: v for k, v in case.items() if k in ("hw", "cin", "c", "S", "d", "heads", "ffn", "nlayers")}
    return make(B=B, M=M, **sizes)


class _Round:
    """A built stage and the buffers of one round: what a training program holds between mini-batches."""

    def __init__(self, case, seed):
        cfg = self.cfg = _config(case)
        B, M, self.K = cfg.B, cfg.M, case["K"]
        dev = torch.device("cuda")
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32

        def normal(shape, scale):
            return [torch.randn(shape, generator=g, device=dev).mul_(scale).to(dt) for _ in range(M)]

        # One buffer per micro-batch.  Activations are of order one; the next stage hands back the gradient of a
        # loss that is a mean, so it is of the order of one over the number of outputs of the mini-batch.
        self.x = normal(gen.boundary_shape(cfg.layout, cfg.in_shape, B), 1.0)
        out = gen.out_shape(cfg.layers, cfg.in_shape)
        if cfg.loss_tail:
            self.labels = [torch.randint(0, out[0], (B,), generator=g, device=dev, dtype=torch.int32) for _ in range(M)]
            self.y = [torch.empty((B,) + tuple(out), device=dev) for _ in range(M)]
            self.loss = [torch.empty(1, device=dev) for _ in range(M)]
            self.dy = [None] * M
        else:
            shape = gen.boundary_shape(cfg.layout, out, B)
            self.dy = normal(shape, 1.0 / (M * math.prod(shape)))
            self.y = [torch.empty(shape, device=dev, dtype=dt) for _ in range(M)]
            self.labels = self.loss = [None] * M
        self.dx = [torch.empty_like(t) if cfg.needs_input_grad else None for t in self.x]

        # Initial weights; the BatchNorm that ends a residual branch starts at a small scale, as deep residual
        # networks are trained.
        weights = []
        ends, shortcut = set(), False
        for i, L in enumerate(cfg.layers):
            if L["kind"] == "res_swap" or (L["kind"] == "res_add" and not shortcut):
                ends.add(i - 1)
            shortcut = L["kind"] == "res_swap" or (shortcut and L["kind"] != "res_add")
        for i, _, shape, fan_in, role in gen.param_specs(cfg.layers):
            n = math.prod(shape)
            if role == "weight":
                std = math.sqrt(2.0 / fan_in) if cfg.init == "kaiming" else 0.02
                weights.append(torch.randn(n, generator=g, device=dev).mul_(std))
            elif role == "gamma":
                small = i in ends and cfg.layers[i]["kind"] == "batchnorm2d"
                weights.append(torch.full((n,), BRANCH_SCALE if small else 1.0, device=dev))
            else:
                weights.append(torch.zeros(n, device=dev))
        self.stage = asteroid.Stage(cfg.layers, B, M, self.K, cfg.in_shape, cfg.dtype, cfg.layout,
                                    cfg.needs_input_grad, stream=torch.cuda.current_stream().cuda_stream)
        self.stage.set_params(torch.cat(weights).cpu().numpy())
        self.fwd_stream = None
        if case["fwd"]:
            self.fwd_stream = asteroid.stream_create()
            self.stage.set_forward_stream(self.fwd_stream)
        self.backward = self.stage.backward_static if case["static"] else self.stage.backward
        self.velocity = torch.empty(self.stage.num_params, pin_memory=True)
        self.velocity_ptr = ctypes.cast(self.velocity.data_ptr(), ctypes.POINTER(ctypes.c_float))

    def __del__(self):
        if getattr(self, "stage", None) is not None:
            self.stage.close()
            if self.fwd_stream:
                asteroid.stream_destroy(self.fwd_stream)


def prepare(case, seed):
    return _Round(case, seed)


def run(state):
    s, st = state, state.stage
    M, K = s.cfg.M, s.K
    for m in range(min(K, M)):
        st.forward(m, s.x[m], s.labels[m], s.y[m], s.loss[m])
    for m in range(M):
        s.backward(m, s.dy[m], s.dx[m])
        if m + K < M:
            st.forward(m + K, s.x[m + K], s.labels[m + K], s.y[m + K], s.loss[m + K])
    st.step(LR, MOMENTUM)
    if st.lib.asteroid_stage_get_velocity(st.h, s.velocity_ptr):
        raise RuntimeError(st.lib.asteroid_last_error().decode())
    return {"y": s.y, "dx": s.dx, "loss": s.loss, "velocity": s.velocity}


def work(case):
    """Boundary tensors once; parameters and velocity read and written by the update and the velocity read back;
    the multiply-adds of the forward pass, of the parameter gradients and of the input gradients."""
    cfg = _config(case)
    shapes = [tuple(cfg.in_shape)] + gen.layer_shapes(cfg.layers, cfg.in_shape)
    n, es = cfg.B * cfg.M, 2 if cfg.dtype == "bf16" else 4
    macs, first, shape = 0, 0, shapes[0]
    for L, o in zip(cfg.layers, shapes[1:]):
        k, here = L["kind"], 0
        if k == "conv2d":
            here = o[1] * o[2] * L["cout"] * (L["cin"] // L["groups"]) * L["k"] ** 2
        elif k == "linear":
            here = math.prod(o) * L["cin"]
        elif k == "mha":
            here = shape[0] * L["d"] * (4 * L["d"] + 2 * shape[0])
        macs += 3 * here
        first = first or here
        shape = o
    if not cfg.needs_input_grad:
        macs -= first
    x, y = math.prod(shapes[0]), math.prod(shapes[-1])
    boundary = n * (x * es * (2 if cfg.needs_input_grad else 1) + (y * 4 if cfg.loss_tail else 2 * y * es))
    return {"bytes": boundary + 20 * gen.num_params(cfg.layers), "flops": 2.0 * macs * n}


def tolerance(case):
    """About four times what the outputs of two rounds differ by when the samples of every micro-batch are permuted
    (every sum over samples in another order), and for bf16 twice what one round differs by from sums in 64 bits
    with the same storage roundings.  Measured (largest over the cases and draws): EfficientNet stage 5e-7, whole model
    7e-5; the ReLU families 4e-3, with single values off by up to 0.8: a value at the edge of a ReLU falls on the other
    side of it, and the gradient behind it appears or vanishes.  bf16: 1e-2 in the convolutions' gradients (the same,
    and the maximum of a pooling window changes place), 9e-3 in the transformer's."""
    if case["family"] in ("vgg", "bert"):
        return {"rel": 2e-2, "max": 0.95}
    if case["family"] in ("effnet", "effnet_full"):
        return {"rel": 2e-4 if case["family"] == "effnet_full" else 5e-6, "max": 2e-2}
    return {"rel": 1e-2, "max": 0.95}
