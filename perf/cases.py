"""What a user has this library do, as timed cases: steady-state steps of single pipeline stages through
`runner.GpuStage`, and whole pipelines emulated on one GPU through `runner.GpuPipeline`.

One pass of a stage case is one mini-batch in the steady state of the nF1B schedule: the single backward pass of the
oldest mini-batch in flight (with real staleness), the fused update / blend / stash write, and the n micro-batch
forwards of the mini-batch that enters; the last stage of a pipeline runs forwards, loss, backward pass and update of
the same mini-batch.  One pass of a pipeline case is a short training run from the first forward to the last update.

The ranges (`draw`), on which the listed cases are points:
  pipe    2 .. 4 stages of a ReLU MLP, width 64 .. 512, micro-batches of 8 .. 64 samples, all five weight policies,
          fp32 and bf16: launches and host time decide
  mlp     two dense layers, width 64 .. 4096 (multiples of 64, of 8, and odd), micro-batches of 16 .. 512 samples,
          interior, first and last stages (logits + softmax cross-entropy), bf16 (fp32 up to width 2048)
  vgg     two 3x3 convolutions and a pooling, twice, from 3 channels, images of 16 .. 64 pixels, bf16 and fp32
  resnet  the four stages of a bottleneck net on 32 .. 128 pixel images: {7x7 stem, conv2_x}, {conv3_x}, {conv4_x},
          {conv5_x, average pooling, classifier + loss}, full or reduced width, bf16 and fp32
  tfm     decoder blocks, model width 256 .. 2048, heads 64 or 128 wide, 32 .. 1024 tokens (whole tiles and not), bf16
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2509_23241_amd import binding as B
from paper_2509_23241_amd.runner import GpuPipeline, GpuStage

DEVICE = "cuda:0"
STAGES = 4                       # stages of the pipeline a single stage is cut from
LAMBDA, MOMENTUM, LR = 0.1, 0.9, 0.01


# ---- the cases -----------------------------------------------------------------------------------------------------

def _pipe(stages, width, mb, n, policy, dtype, minibatches=8):
    return dict(kind="pipe", stages=stages, width=width, mb=mb, n=n, policy=policy, dtype=dtype, minibatches=minibatches)


def _mlp(width, stage, mb, n, act, policy, dtype, classes=0):
    return dict(kind="mlp", width=width, stage=stage, mb=mb, n=n, act=act, policy=policy, dtype=dtype, classes=classes)


def _vgg(size, channels, mb, n, policy, dtype):
    return dict(kind="vgg", size=size, channels=channels, stage=0, mb=mb, n=n, policy=policy, dtype=dtype)


def _resnet(stage, size, channels, identity, mb, n, policy, dtype):
    return dict(kind="resnet", stage=stage, size=size, channels=channels, identity=identity, mb=mb, n=n, policy=policy,
                dtype=dtype)


def _tfm(d, head, tokens, blocks, mb, n, policy):
    return dict(kind="tfm", d=d, head=head, tokens=tokens, blocks=blocks, stage=1, mb=mb, n=n, policy=policy, dtype="bf16")


def listed():
    return [
        # the smallest training run: 256-512-512-10 in fp32 on two stages, eight mini-batches
        dict(_pipe(2, 256, 32, 4, "convex", "f32"), name="pipe_f32_256"),
        # a small interior stage that keeps no stash (V-TiMePReSt)
        dict(_mlp(512, 1, 64, 4, "relu", "latest", "bf16"), name="mlp_bf16_512"),
        # the configuration the headline figure is quoted on
        dict(_mlp(4096, 1, 256, 8, "gelu", "convex", "bf16"), name="mlp_bf16_4096"),
        # a last stage with 1000 classes at sizes that fill no tile
        dict(_mlp(2000, 3, 100, 4, "gelu", "stashed", "bf16", classes=1000), name="mlp_bf16_2000_loss"),
        # single precision, as the smallest configuration trains, at an ordinary width
        dict(_mlp(1024, 1, 128, 4, "relu", "eq1", "f32"), name="mlp_f32_1024"),
        # first stage of the VGG-16-style net on 32x32 images, in bf16 and in single precision
        dict(_vgg(32, 64, 64, 4, "convex", "bf16"), name="vgg_bf16_32px"),
        dict(_vgg(32, 64, 16, 2, "convex", "f32"), name="vgg_f32_32px"),
        # the bottleneck net on 64x64 images: stem and conv2_x; conv4_x; conv5_x, pooling, 200 classes and loss
        dict(_resnet(0, 64, 64, 2, 128, 4, "convex", "bf16"), name="resnet_bf16_stem"),
        dict(_resnet(2, 64, 64, 5, 128, 4, "convex", "bf16"), name="resnet_bf16_conv4"),
        dict(_resnet(3, 64, 64, 2, 128, 4, "convex", "bf16"), name="resnet_bf16_head"),
        # a decoder block at the size of the transformer configuration (32 sequences of 1024 tokens)
        dict(_tfm(2048, 128, 1024, 1, 8, 4, "convex"), name="tfm_bf16_2048"),
        # a small decoder on sequences that are not whole tiles
        dict(_tfm(512, 64, 200, 2, 8, 4, "convex"), name="tfm_bf16_512_ragged"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi):
    """Half the widths are multiples of 64, a quarter multiples of 8, a quarter anything."""
    w = _log(rng, lo, hi)
    unit = rng.choice([64, 64, 8, 1])
    return min(max(unit, int(round(w / unit)) * unit), hi)


def _draw_once(rng):
    kind = rng.choice(["mlp", "mlp", "mlp", "pipe", "vgg", "resnet", "resnet", "tfm", "tfm"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    policy = rng.choice(["convex", "convex", "eq1", "stashed", "latest"])
    n = rng.choice([1, 2, 3, 4, 4, 8])
    mb = int(round(_log(rng, 16, 512)))
    if rng.random() < 0.6:
        mb = max(8, mb // 8 * 8)
    if kind == "pipe":
        return _pipe(rng.randint(2, STAGES), _width(rng, 64, 512), min(mb, 64), max(n, 2),
                     rng.choice([policy, "timeprest"]), dtype, rng.randint(6, 10))
    if kind == "mlp":
        stage = rng.randrange(STAGES)
        classes = rng.choice([10, 100, 200, 1000]) if stage == STAGES - 1 else 0
        return _mlp(_width(rng, 64, 2048 if dtype == "f32" else 4096), stage, mb, n, rng.choice(["gelu", "relu"]), policy,
                    dtype, classes)
    mb = max(16 if kind == "resnet" else 4, mb // 4)
    if kind == "vgg":
        return _vgg(rng.choice([16, 20, 24, 28, 32, 32, 48, 64]), rng.choice([32, 48, 64, 64]), mb, n, policy, dtype)
    if kind == "resnet":
        return _resnet(rng.randrange(STAGES), rng.choice([32, 64, 64, 96, 128]), rng.choice([16, 32, 64, 64]),
                       rng.randint(1, 5), mb, n, policy, dtype)
    d = rng.choice([256, 384, 512, 768, 1024, 1536, 2048])
    tokens = rng.choice([32, 64, 128, 256, 512, 1024, int(_log(rng, 32, 1024))])
    return _tfm(d, rng.choice([64, 64, 128]), tokens, rng.randint(1, 2), max(1, mb // 8), n, policy)


def draw(rng):
    """Sizes are redrawn until the case's work fits: fp32, and image sizes that are no power of two, leave a smaller
    share of the largest listed case's operations, since they run further from the matrix cores' bf16 rate."""
    while True:
        c = _draw_once(rng)
        limit = 1.2e12
        if c["dtype"] == "f32":
            limit = 2e10
        elif c.get("size", 1) & (c.get("size", 1) - 1):
            limit = 3e10
        elif c["kind"] == "tfm" and c["tokens"] % 64:
            limit = 2e11
        if 1e6 < work(c)["flops"] <= limit:
            return c


# ---- layers, in the tuple format of runner.GpuStage ----------------------------------------------------------------

def _bottleneck(cin, mid, cout, h, stride, first):
    t, ho = h * h, h // stride
    to = ho * ho
    out = [("res", cin, t, "begin"), (cin, mid, "none", t), ("bn", mid, t, "relu"),
           ("conv", mid, mid, h, h, "none", stride, 3), ("bn", mid, to, "relu"), (mid, cout, "none", to),
           ("bn", cout, to, "none")]
    if first:
        out.append(("swap", cout, to, cin, t))
        if stride == 2:
            out.append(("sub", cin, h, h))
        out += [(cin, cout, "none", to), ("bn", cout, to, "none")]
    out.append(("res", cout, to, "add", "relu"))
    return out


def _layers(c):
    kind = c["kind"]
    if kind == "mlp":
        w = c["width"]
        return [(w, w, c["act"]), (w, c["classes"], "none") if c["classes"] else (w, w, c["act"])]
    if kind == "vgg":
        s, a, b = c["size"], c["channels"], 2 * c["channels"]
        return [("conv", 3, a, s, s, "relu"), ("conv", a, a, s, s, "relu"), ("pool", a, s, s),
                ("conv", a, b, s // 2, s // 2, "relu"), ("conv", b, b, s // 2, s // 2, "relu"), ("pool", b, s // 2, s // 2)]
    if kind == "resnet":
        s, g = c["stage"], c["channels"]
        h = c["size"] // 4
        out = []
        if s == 0:
            out += [("conv", 3, g, c["size"], c["size"], "none", 2, 7), ("bn", g, 4 * h * h, "relu"), ("pool", g, 2 * h, 2 * h)]
            cin, mid, stride = g, g, 1
        else:
            cin, mid, stride = g * 2 ** (s + 1), g * 2 ** s, 2
            h >>= s - 1
        out += _bottleneck(cin, mid, 4 * mid, h, stride, True)
        for _ in range(c["identity"]):
            out += _bottleneck(4 * mid, mid, 4 * mid, h // stride, 1, False)
        if s == 3:
            out += [("avg", 4 * mid, (h // 2) ** 2), (4 * mid, 200, "none")]
        return out
    d, t = c["d"], c["tokens"]
    block = [("res", d, t, "begin"), ("ln", d, t), (d, 3 * d, "none", t), ("attn", d, d // c["head"], t), (d, d, "none", t),
             ("res", d, t, "add"), ("res", d, t, "begin"), ("ln", d, t), (d, 4 * d, "gelu", t), (4 * d, d, "none", t),
             ("res", d, t, "add")]
    return block * c["blocks"]


def _pipe_stages(c):
    """The layers of a pipeline w-2w-2w-10 (two stages: the first two layers, then the last), one more 2w-2w layer for
    every further stage."""
    w, k = c["width"], c["stages"]
    stages = [[(w, 2 * w, "relu"), (2 * w, 2 * w, "relu")]] + [[(2 * w, 2 * w, "relu")] for _ in range(k - 2)]
    return stages + [[(2 * w, 10, "none")]]


def _is_last(c):
    return c["stage"] == STAGES - 1


def _layer_flops(l):
    """Multiply-adds of one sample's forward pass, times two."""
    if l[0] == "conv":
        stride, k = (l[6], l[7]) if len(l) > 6 else (1, 3)
        return 2 * (l[3] // stride) * (l[4] // stride) * l[2] * k * k * l[1]
    if l[0] == "attn":
        return 2 * l[3] * l[3] * l[1]      # two products over half of the scores
    if isinstance(l[0], str):
        return 0
    return 2 * l[0] * l[1] * (l[3] if len(l) > 3 else 1)


def _params(layers):
    return sum(int(np.prod(s)) for l in layers for s in B.layer_param_shapes(l))


def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    rows = c["mb"] * c["n"]
    if c["kind"] == "pipe":
        stages = _pipe_stages(c)
        flops = sum(3 * _layer_flops(l) for s in stages for l in s) * rows * c["minibatches"]
        # weights and momentum in and out once per update, the input once
        nbytes = c["minibatches"] * (16 * sum(_params(s) for s in stages) + rows * c["width"] * es)
        return {"bytes": nbytes, "flops": flops}
    layers = _layers(c)
    flops = 0
    for i, l in enumerate(layers):
        f = _layer_flops(l)
        # forward, gradient of the weights, gradient of the input (none at the first layer of the first stage);
        # attention's backward pass has five products for two forward
        flops += f * (3.5 if l[0] == "attn" else 2 if i == 0 and c["stage"] == 0 else 3)
    ins, outs = B.layer_in_elems(layers[0]), B.layer_out_elems(layers[-1])
    acts = rows * es * (ins * (2 if c["stage"] > 0 else 1) + outs * 2)     # x, y, dy (or dlogits), dx
    stale = c["policy"] != "latest" and not _is_last(c)
    # per parameter: latest weights, momentum in; weights, momentum, gradient out; the stashed version in
    return {"bytes": acts + _params(layers) * (24 if stale else 20), "flops": flops * rows}


# Largest relative difference of any returned tensor between two correct executions of a case.  Measured, per kind and
# precision: the fp32 biases and normalisation shifts were moved by 1e-6 (bf16 cases) or 3e-7 (fp32 cases), which is what
# sums in another order do to a pre-activation, and the outputs of the two runs compared; stated is about four times
# the largest difference seen.  In bf16 the moved sums round to other neighbours here and there (2e-3 on dense layers,
# 1.2e-2 through two decoder blocks); ReLU masks and pooling windows decided by such a rounding add to it (1.1e-2
# through the VGG stage, 4.5e-2 through six bottlenecks with batch normalisation).
_REL = {("pipe", "f32"): 1e-5, ("mlp", "f32"): 1e-5, ("vgg", "f32"): 5e-4, ("resnet", "f32"): 2e-3,
        ("pipe", "bf16"): 1e-2, ("mlp", "bf16"): 1e-2, ("vgg", "bf16"): 5e-2, ("resnet", "bf16"): 0.16, ("tfm", "bf16"): 5e-2}


def tolerance(case):
    return {"rel": _REL[case["kind"], case["dtype"]]}


# ---- inputs --------------------------------------------------------------------------------------------------------

class _Draws:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(seed)

    def normal(self, shape, std=1.0):
        return torch.randn(shape, generator=self.gen, device=DEVICE) * std

    def labels(self, rows, classes):
        return torch.randint(0, classes, (rows,), generator=self.gen, device=DEVICE, dtype=torch.int32)

    def params(self, layers):
        """Initial parameters as the list of arrays GpuStage takes.  In front of a ReLU the shifts (biases, shifts of
        normalisations) are about three standard deviations of the pre-activation, up in every second channel and down in
        the others, and weights are scaled so that activations keep a mean square of one: half of the activations are
        zeros, as behind any ReLU, but few pre-activations lie so near zero that a rounding error decides their sign, and
        gradients of two executions can be compared."""
        out = []
        for i, l in enumerate(layers):
            shapes = B.layer_param_shapes(l)
            if not shapes:
                continue
            channels = shapes[1][0]
            side = torch.ones(channels, device=DEVICE)
            side[1::2] = -1
            shift = self.normal(channels, 0.02)
            following = layers[i + 1] if i + 1 < len(layers) else ("end",)
            if l[0] in ("ln", "bn"):
                w = torch.ones(channels, device=DEVICE)
                if l[0] == "bn" and l[3] == "relu":
                    shift += 3 * side
                elif l[0] == "bn" and (following[0] == "swap" or layers[i - 2][0] in ("sub", "swap")):
                    shift += 1.5 * side          # the two branches of a block that changes the number of channels
                elif l[0] == "bn":
                    shift += 0.7 * side - 1.0    # adds to an activation that is zero already in every second channel
                    shift[0::2] += 1.0
            else:
                act = l[5] if l[0] == "conv" else l[2]
                w = self.normal(shapes[0], math.sqrt((0.2 if act == "relu" else 2.0) / np.prod(shapes[0][1:])))
                if act == "relu":
                    shift += 1.35 * side
            out += [w.cpu().numpy(), shift.cpu().numpy()]
        return out


def _spec(l):
    return SimpleNamespace(in_features=l[0], out_features=l[1], act=l[2])


class _Pipeline:
    def __init__(self, c, seed):
        g = _Draws(seed)
        stages = _pipe_stages(c)
        w = SimpleNamespace(stages=[[_spec(l) for l in s] for s in stages], K=len(stages), dtype=c["dtype"], mb=c["mb"],
                            n=c["n"], lam=LAMBDA, lr=LR, momentum=MOMENTUM)
        self.pipe = GpuPipeline(w, [g.params(s) for s in stages], policy=c["policy"], device=DEVICE)
        self.minibatches, self.timeprest = c["minibatches"], c["policy"] == "timeprest"
        rows = c["mb"] * c["n"]
        dtype = self.pipe.stages[0].tdtype
        self.x = [g.normal((rows, c["width"])).to(dtype) for _ in range(self.minibatches)]
        self.labels = [g.labels(rows, 10) for _ in range(self.minibatches)]

    def run(self):
        drive = self.pipe.run_microbatches if self.timeprest else self.pipe.run
        _, losses = drive(self.minibatches, self.x.__getitem__, self.labels.__getitem__)
        out = {"losses": [losses[j] for j in range(self.minibatches)]}
        for k, st in enumerate(self.pipe.stages):
            out["weights%d" % k], out["momentum%d" % k] = _latest(st), st.momentum
        return out


def _latest(st):
    """The latest weights where they lie in the stage's ring."""
    slot = int(st.query().latest_version) % st.C
    return st.ring[slot * st.P:(slot + 1) * st.P]


class _Stage:
    """A stage in its steady state.  Mini-batches take turns on two inputs; every eighth mini-batch the upstream
    gradients change sign (at a last stage the labels change), so that thousands of passes neither walk the weights
    away nor learn the inputs by heart."""

    def __init__(self, c, seed):
        g = _Draws(seed)
        layers = _layers(c)
        self.c, self.rows = c, c["mb"] * c["n"]
        self.last, self.depth = _is_last(c), STAGES - c["stage"]
        streams = 0 if c["kind"] == "tfm" else 3 if self.last else 2
        self.st = st = GpuStage(layers, g.params(layers), dtype=c["dtype"], mb=c["mb"], n=c["n"], stage_index=c["stage"],
                                num_stages=STAGES, policy=c["policy"], lam=LAMBDA, lr=LR, momentum=MOMENTUM,
                                device=DEVICE, forward_stream=streams)
        self.x = [g.normal((self.rows, st.in_elems)).to(st.tdtype) for _ in range(2)]
        if self.last:
            self.labels = [g.labels(self.rows, st.out_elems) for _ in range(4)]
        else:
            dy = [g.normal((self.rows, st.out_elems), 1 / (math.sqrt(st.out_elems) * self.rows)).to(st.tdtype) for _ in range(2)]
            self.dy = dy + [-d for d in dy]
        self.y = torch.empty(self.rows, st.out_elems, dtype=st.tdtype, device=DEVICE)
        self.dx = torch.empty(self.rows, st.in_elems, dtype=st.tdtype, device=DEVICE) if st.needs_dx else None
        self.j = 0
        if not self.last:
            for j in range(self.depth):
                self.forward(j)
            for _ in range(self.depth):      # to the steady staleness
                self.run()

    def forward(self, j):
        x, y, mb = self.x[j % 2], self.y, self.c["mb"]
        for ub in range(self.c["n"]):
            self.st.forward(j, ub, x[ub * mb:(ub + 1) * mb], y[ub * mb:(ub + 1) * mb])

    def run(self):
        st, j = self.st, self.j
        self.j += 1
        out = {"y": self.y, "gradient": st.grad, "momentum": st.momentum}
        if self.last:
            self.forward(j)
            out["loss"], out["dlogits"] = st.loss(j, self.y, self.labels[j // 8 % 2 * 2 + j % 2])
            st.backward(j, out["dlogits"], self.dx)
            st.blend_update(j)
        else:
            st.backward(j, self.dy[j // 8 % 2 * 2 + j % 2], self.dx)
            st.blend_update(j, j + 1)
            self.forward(j + self.depth)
        out["weights"] = _latest(st)
        if self.dx is not None:
            out["dx"] = self.dx
        return out


def prepare(case, seed):
    return _Pipeline(case, seed) if case["kind"] == "pipe" else _Stage(case, seed)


def run(state):
    return state.run()
