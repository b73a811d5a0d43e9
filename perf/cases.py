"""Workloads whose speed is tracked: what a user has this library do, through the calls of `binding.py`.

Six kinds of work, each over the range of sizes it meets in use:

  conv        one convolution layer of a training step: forward, backward-data, backward-filter with the bias gradient
  stem        the first layer of an image network (RGB input): forward and backward-filter, no backward-data
  bottleneck  the four convolutions of a residual block that changes resolution: forward and both gradients of each
  pair        a 1xL and an Lx1 convolution in a row: forward and both gradients of each
  dense       one dense layer, forward and backward in one library call
  vgg16       a VGG-16 training step of a given per-GPU batch, all layers and the loss

Everything runs on the current stream.  Single layers run on the library's default kernel choice, with plain calls.  The
VGG-16 step is issued as a training loop issues it: pre-marshalled calls, measured kernel choice (caches flushed).

Inputs are made on the GPU from the seed: images are N(0,1), activations behind a ReLU are max(N(0,1), 0), gradients
that reach a layer through a ReLU are N(0,1) with half of the entries masked, weights are He-normal, biases uniform.
"""
import math

import torch

from paper_2112_10065_amd import binding as dp, workloads

BF16, F32 = "bf16", "f32"


def listed():
    return [
        # the fp32 reference layer: the smallest call, all launch and latency
        dict(name="conv16_f32_n2", kind="conv", n=2, h=16, w=16, c=16, k=16, r=3, stride=1, pad=1, dtype=F32, mask="own", bias=False),
        # a late layer at the batch that 32-way strong scaling leaves: few pixels, many channels, weights dominate
        dict(name="conv14_512_n1", kind="conv", n=1, h=14, w=14, c=512, k=512, r=3, stride=1, pad=1, dtype=BF16, mask="front", bias=True),
        # a middle layer at a middle batch
        dict(name="conv28_512_n8", kind="conv", n=8, h=28, w=28, c=512, k=512, r=3, stride=1, pad=1, dtype=BF16, mask="front", bias=True),
        # an early layer: large image, 64 channels, bound by memory
        dict(name="conv224_64_n16", kind="conv", n=16, h=224, w=224, c=64, k=64, r=3, stride=1, pad=1, dtype=BF16, mask="front", bias=True),
        # channel counts and an image that no tile divides, no padding, mask kept with the layer
        dict(name="conv73_80_192_n4", kind="conv", n=4, h=73, w=73, c=80, k=192, r=3, stride=1, pad=0, dtype=BF16, mask="own", bias=False),
        # the first layer of a residual network at the whole batch
        dict(name="stem7_224_n32", kind="stem", n=32, h=224, w=224, k=64, r=7, stride=2, pad=3, bias=False),
        # the background job of the multiplexing run: the block that enters the second stage at batch 64
        dict(name="bottleneck56_n64", kind="bottleneck", n=64, h=56, w=56, c=256, mid=128, k=512, stride=2),
        # factorised 1x7 / 7x1 convolutions at 17 x 17
        dict(name="pair17_160_192_n16", kind="pair", n=16, h=17, w=17, c=160, mid=160, k=192, length=7),
        # the largest dense layer at a small shard: a stream over the weights
        dict(name="dense25088_n2", kind="dense", n=2, inputs=25088, outputs=4096),
        # training steps: the shards that 16-way and 4-way data parallelism leave (gradients go to the other GPUs next), and
        # the whole batch on one GPU, which also updates its weights
        dict(name="vgg16_n2", kind="vgg16", n=2, image=224, classes=1000, update=False),
        dict(name="vgg16_n8", kind="vgg16", n=8, image=224, classes=1000, update=False),
        dict(name="vgg16_n32_update", kind="vgg16", n=32, image=224, classes=1000, update=True),
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        kind = rng.choice(["conv", "conv", "conv", "conv_any", "conv_f32", "stem", "bottleneck", "pair", "dense", "vgg16", "vgg16"])
        if kind == "conv":      # 3x3 layers of the VGG / residual kind: channels in whole 64s, image from 7 to 224
            h = _spread(rng, 7, 224)
            c, k = 64 * _spread(rng, 1, 8), 64 * _spread(rng, 1, 8)
            case = dict(kind=kind, n=_spread(rng, 1, 32), h=h, w=h + rng.randint(-h // 8, h // 8), c=c, k=k, r=3, stride=1, pad=1, dtype=BF16,
                        mask=rng.choice(["front", "front", "own"]), bias=rng.random() < 0.7)
        elif kind == "conv_any":  # channels in whole 16s, unit or double stride, with and without padding
            h = _spread(rng, 8, 150)
            case = dict(kind="conv", n=_spread(rng, 1, 16), h=h, w=h, c=16 * rng.randint(2, 28), k=16 * rng.randint(2, 28), r=rng.choice([1, 3, 3, 5]),
                        stride=rng.choice([1, 1, 2]), pad=rng.choice([0, 1]), dtype=BF16, mask=rng.choice(["front", "own"]), bias=False)
        elif kind == "conv_f32":  # small layers in the reference precision
            h = rng.randint(8, 40)
            case = dict(kind="conv", n=rng.randint(1, 4), h=h, w=h, c=rng.randint(4, 64), k=rng.randint(4, 64), r=3, stride=1, pad=1, dtype=F32,
                        mask="own", bias=rng.random() < 0.5)
        elif kind == "stem":
            r = rng.choice([3, 7])
            stride = 2 if r == 7 else rng.choice([1, 2])
            h = rng.randint(150, 400)
            case = dict(kind=kind, n=_spread(rng, 1, 32), h=h, w=h, k=rng.choice([32, 64]), r=r, stride=stride, pad=r // 2 if stride == 1 or r == 7 else 0,
                        bias=rng.random() < 0.5)
        elif kind == "bottleneck":
            mid = 64 * _spread(rng, 1, 8)
            h = _spread(rng, 7, 100)
            stride = rng.choice([1, 2])
            case = dict(kind=kind, n=_spread(rng, 1, 64), h=h, w=h, c=mid * rng.choice([1, 2, 4]), mid=mid, k=4 * mid, stride=stride)
        elif kind == "pair":
            h = rng.randint(8, 35)
            case = dict(kind=kind, n=_spread(rng, 1, 32), h=h, w=h, c=32 * rng.randint(3, 14), mid=32 * rng.randint(3, 14), k=32 * rng.randint(3, 14),
                        length=rng.choice([3, 7]))
        elif kind == "dense":
            case = dict(kind=kind, n=_spread(rng, 1, 32), inputs=64 * _spread(rng, 8, 392), outputs=8 * _spread(rng, 16, 512))
        else:
            n = _spread(rng, 1, 32)
            case = dict(kind=kind, n=n, image=32 * rng.randint(3, 7), classes=rng.choice([100, 200, 365, 1000]), update=rng.random() < 0.3)
        if kind == "vgg16" or work(case)["flops"] <= 8e11 and work(case)["bytes"] <= 4e9:
            return case


# ---- shapes -------------------------------------------------------------------------------------------------------

def _conv_layers(case):
    """The convolutions of a case as (h, w, c, k, r, s, stride, (pad_h, pad_w)), in order."""
    kind = case["kind"]
    if kind == "conv":
        return [(case["h"], case["w"], case["c"], case["k"], case["r"], case["r"], case["stride"], (case["pad"], case["pad"]))]
    if kind == "stem":
        return [(case["h"], case["w"], 3, case["k"], case["r"], case["r"], case["stride"], (case["pad"], case["pad"]))]
    if kind == "bottleneck":
        h, w, c, m, k, st = (case[x] for x in ("h", "w", "c", "mid", "k", "stride"))
        h2, w2 = (h + 2 - 3) // st + 1, (w + 2 - 3) // st + 1
        return [(h, w, c, m, 1, 1, 1, (0, 0)), (h, w, m, m, 3, 3, st, (1, 1)), (h2, w2, m, k, 1, 1, 1, (0, 0)), (h, w, c, k, 1, 1, st, (0, 0))]
    if kind == "pair":
        h, w, p = case["h"], case["w"], case["length"] // 2
        return [(h, w, case["c"], case["mid"], 1, case["length"], 1, (0, p)), (h, w, case["mid"], case["k"], case["length"], 1, 1, (p, 0))]
    raise ValueError(kind)


def _out(layer):
    h, w, _, _, r, s, st, (ph, pw) = layer
    return (h + 2 * ph - r) // st + 1, (w + 2 * pw - s) // st + 1


def _vgg16(case):
    """[("conv", hw, c, k, pool behind it) ..., ("dense", inputs, outputs, relu) ...]"""
    convs = workloads.vgg16_convs()
    ops, hw = [], case["image"]
    for i, l in enumerate(convs):
        pool = i + 1 == len(convs) or convs[i + 1].h != l.h
        ops.append(("conv", hw, l.c, l.k, pool))
        hw = hw // 2 if pool else hw
    width = workloads.vgg16_linears()[0].out_f
    sizes = [hw * hw * convs[-1].k, width, width, case["classes"]]
    return ops + [("dense", sizes[i], sizes[i + 1], i < 2) for i in range(3)]


# ---- inputs -------------------------------------------------------------------------------------------------------

class _Gen:
    def __init__(self, seed):
        self.dev = torch.device("cuda:0")
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(int(seed))

    def normal(self, shape, dtype, scale=1.0, relu=False, masked=False):
        t = torch.randn(shape, generator=self.gen, device=self.dev, dtype=torch.float32)
        if scale != 1.0:
            t *= scale
        if relu:
            t.relu_()
        if masked:
            t *= torch.rand(shape, generator=self.gen, device=self.dev) < 0.5
        return t.to(dtype)

    def bias(self, k):
        return torch.rand(k, generator=self.gen, device=self.dev) * 0.2 - 0.1

    def empty(self, shape, dtype):
        return torch.empty(shape, device=self.dev, dtype=dtype)

    def workspace(self, nbytes):
        return torch.empty(max(int(nbytes), 256), device=self.dev, dtype=torch.uint8)


class _ConvLayer:
    """One convolution with everything its three calls take."""

    def __init__(self, g, n, layer, dtype, mask, bias, first=False):
        h, w, c, k, r, s, st, pad = layer
        ho, wo = _out(layer)
        t = torch.bfloat16 if dtype == BF16 else torch.float32
        flags = (dp.DP_BIAS if bias else 0) | dp.DP_RELU | (dp.DP_RELU_IN if mask == "front" else 0)
        self.desc = dp.conv_desc(n, h, w, c, k, r, s, (st, st), pad, dp.DP_BF16 if dtype == BF16 else dp.DP_F32, flags)
        self.first, self.mask = first, mask
        self.x = g.normal((n, h, w, c), t, relu=mask == "front")
        self.wt = g.normal((k, r, s, c), t, scale=math.sqrt(2.0 / (r * s * c)))
        self.bias = g.bias(k) if bias else None
        # with the mask in front (DP_RELU_IN) the incoming gradient has been masked by the layer behind
        self.dy = g.normal((n, ho, wo, k), t, masked=mask == "front")
        self.y = g.empty((n, ho, wo, k), t)
        self.dx = None if first else g.empty((n, h, w, c), t)
        self.dw, self.db = g.empty((k, r, s, c), torch.float32), g.empty((k,), torch.float32)
        self.ws = g.workspace(max(dp.dp_conv2d_workspace_bytes(self.desc, p) for p in range(3)))

    def run(self):
        dp.dp_conv2d_fwd(self.desc, self.x, self.wt, self.bias, self.y, self.ws)
        saved = self.y if self.mask == "own" else None
        if not self.first and self.mask == "front":
            dp.dp_conv2d_bwd_data_relu(self.desc, self.dy, None, self.wt, self.x, self.dx, self.ws)
        elif not self.first:
            dp.dp_conv2d_bwd_data(self.desc, self.dy, saved, self.wt, self.dx, self.ws)
        dp.dp_conv2d_bwd_filter(self.desc, self.x, self.dy, saved, self.dw, self.db, self.ws)
        return [t for t in (self.y, self.dx, self.dw, self.db) if t is not None]


class _Layers:
    """Layers run one after another, each on its own tensors."""

    def __init__(self, layers):
        self.layers = layers

    def run(self):
        return [l.run() for l in self.layers]


class _Dense:
    def __init__(self, g, n, inputs, outputs):
        t = torch.bfloat16
        self.desc = dp.linear_desc(n, inputs, outputs, dp.DP_BF16, dp.DP_BIAS | dp.DP_RELU | dp.DP_RELU_IN)
        self.x = g.normal((n, inputs), t, relu=True)
        self.wt = g.normal((outputs, inputs), t, scale=math.sqrt(2.0 / inputs))
        self.bias, self.dy = g.bias(outputs), g.normal((n, outputs), t, masked=True)
        self.y, self.dx = g.empty((n, outputs), t), g.empty((n, inputs), t)
        self.dw, self.db = g.empty((outputs, inputs), torch.float32), g.empty((outputs,), torch.float32)
        self.ws = g.workspace(dp.dp_linear_workspace_bytes(self.desc))

    def run(self):
        dp.dp_linear_fwd_bwd(self.desc, x=self.x, W=self.wt, bias=self.bias, dy=self.dy, y=self.y, dx=self.dx, dW=self.dw, dbias=self.db, ws=self.ws)
        return [self.y, self.dx, self.dw, self.db]


class _Vgg16Step:
    """One training step over the 21 layers of VGG-16 and the loss, layer by layer: every layer works on resident tensors of its
    own (so that no rounding is handed on from layer to layer and each output can be compared); with `update` the SGD step
    follows.  Weights, gradients, momentum, outputs and input gradients are flat buffers, the layers use slices of them."""

    def __init__(self, g, case):
        n, bf, f32 = case["n"], torch.bfloat16, torch.float32
        ops = _vgg16(case)
        dp.dp_set_autotune(2)
        conv = [o[0] == "conv" for o in ops]
        wide = [9 * o[2] * o[3] if c else o[1] * o[2] for o, c in zip(ops, conv)]           # weights
        outs = [o[3] if c else o[2] for o, c in zip(ops, conv)]                             # biases
        x_shape = [(n, o[1], o[1], o[2]) if c else (n, o[1]) for o, c in zip(ops, conv)]
        y_shape = [(n, o[1], o[1], o[3]) if c else (n, o[2]) for o, c in zip(ops, conv)]

        def slices(sizes, dtype):
            """A flat buffer and one slice per size, each at a whole 16-byte unit."""
            at = [0]
            for s in sizes:
                at.append(at[-1] + (s + 7) // 8 * 8)
            flat = torch.zeros(at[-1], device=g.dev, dtype=dtype)
            return flat, [flat[at[i]:at[i] + s] for i, s in enumerate(sizes)]

        self.w32, w32 = slices(wide, f32)
        self.b32, b32 = slices(outs, f32)
        for i, o in enumerate(ops):
            w32[i].copy_(g.normal((wide[i],), f32, scale=math.sqrt(2.0 / (9 * o[2] if conv[i] else o[1]))))
            b32[i].copy_(g.bias(outs[i]))
        self.w16, w16 = slices(wide, bf)
        self.w16.copy_(self.w32)
        self.dw, dw = slices(wide, f32)
        self.db, db = slices(outs, f32)
        self.y, y = slices([math.prod(s) for s in y_shape], bf)
        self.dx, dx = slices([math.prod(s) for s in x_shape[1:]], bf)
        dx = [None] + dx                                     # a training step never uses the gradient of the image
        x = [g.normal(s, bf, relu=i > 0) for i, s in enumerate(x_shape)]
        dy = [g.normal(s, bf, masked=i + 1 < len(ops)) for i, s in enumerate(y_shape)]
        pooled = [i for i, o in enumerate(ops) if conv[i] and o[4]]
        px = {i: g.normal(y_shape[i], bf, relu=True) for i in pooled}
        half = {i: (n, ops[i][1] // 2, ops[i][1] // 2, ops[i][3]) for i in pooled}
        pdy = {i: g.normal(half[i], bf, masked=True) for i in pooled}
        py, pdx = {i: g.empty(half[i], bf) for i in pooled}, {i: g.empty(y_shape[i], bf) for i in pooled}
        logits = g.normal((n, case["classes"]), bf)
        labels = torch.randint(0, case["classes"], (n,), generator=g.gen, device=g.dev, dtype=torch.int32)
        loss, dlogits = torch.zeros(4, device=g.dev), torch.empty_like(logits)
        self.outputs = {"y": self.y, "dx": self.dx, "dw": self.dw, "db": self.db, "loss": loss[:1], "dlogits": dlogits,
                        "pool_y": list(py.values()), "pool_dx": list(pdx.values())}

        main = torch.cuda.current_stream()
        descs = []
        for i, o in enumerate(ops):
            if conv[i]:
                flags = dp.DP_BIAS | dp.DP_RELU | (dp.DP_RELU_IN if i else 0)
                descs.append(dp.conv_desc(n, o[1], o[1], o[2], o[3], 3, 3, (1, 1), (1, 1), dp.DP_BF16, flags))
            else:
                descs.append(dp.linear_desc(n, o[1], o[2], dp.DP_BF16, dp.DP_BIAS | (dp.DP_RELU if o[3] else 0) | dp.DP_RELU_IN))
        need = max(max(dp.dp_conv2d_workspace_bytes(d, p) for p in range(3)) if c else dp.dp_linear_workspace_bytes(d) for d, c in zip(descs, conv))
        ws = g.workspace(need)

        self.calls = []
        call = lambda name, *a: self.calls.append(dp.bind(name, *a))
        for i, o in enumerate(ops):
            if conv[i]:
                call("dp_conv2d_fwd", descs[i], x[i], w16[i], b32[i], y[i], ws, main)
                if i in px:
                    call("dp_maxpool2x2_fwd", n, o[1], o[1], o[3], dp.DP_BF16, px[i], py[i], main)
            else:
                call("dp_linear_fwd_bwd", descs[i], x[i], w16[i], b32[i], None, None, y[i], None, None, None, ws, main)
        call("dp_softmax_xent", n, case["classes"], dp.DP_BF16, logits, labels, loss, dlogits, main)
        for i in reversed(range(len(ops))):
            o = ops[i]
            if i in px:
                call("dp_maxpool2x2_bwd", n, o[1], o[1], o[3], dp.DP_BF16, px[i], pdy[i], pdx[i], main)
            if conv[i]:
                call("dp_conv2d_bwd_filter", descs[i], x[i], dy[i], None, dw[i], db[i], ws, main)
                if i:
                    call("dp_conv2d_bwd_data_relu", descs[i], dy[i], None, w16[i], x[i], dx[i], ws, main)
            else:
                call("dp_linear_fwd_bwd", descs[i], x[i], None, None, dy[i], None, None, None, dw[i], db[i], ws, main)
                call("dp_linear_fwd_bwd", descs[i], x[i], w16[i], None, dy[i], None, None, dx[i], None, None, ws, main)
        # the measured kernel choice times its candidates here, each call alone on the GPU
        for launch in self.calls:
            launch()
            torch.cuda.synchronize()
        if case["update"]:
            mw, mb = torch.zeros_like(self.dw), torch.zeros_like(self.db)
            call("dp_sgd_update", mw.numel(), 1e-6, 0.9, self.dw, mw, self.w32, self.w16, main)
            call("dp_sgd_update", mb.numel(), 1e-6, 0.9, self.db, mb, self.b32, None, main)
            self.outputs.update(w32=self.w32, w16=self.w16, b32=self.b32, mw=mw, mb=mb)

    def run(self):
        for launch in self.calls:
            launch()
        return self.outputs


def prepare(case, seed):
    g = _Gen(seed)
    dp.dp_set_autotune(0)
    kind, n = case["kind"], case["n"]
    if kind == "vgg16":
        return _Vgg16Step(g, case)
    if kind == "dense":
        return _Dense(g, n, case["inputs"], case["outputs"])
    if kind == "conv":
        return _ConvLayer(g, n, _conv_layers(case)[0], case["dtype"], case["mask"], case["bias"])
    if kind == "stem":      # a first layer's gradient arrives masked when its mask is applied by the layer behind
        return _ConvLayer(g, n, _conv_layers(case)[0], BF16, "none", case["bias"], first=True)
    return _Layers([_ConvLayer(g, n, l, BF16, "front", False) for l in _conv_layers(case)])


def run(state):
    return state.run()


# ---- what a pass cannot do without -------------------------------------------------------------------------------------

def work(case):
    """Each input read once, each output written once; flops of the multiply-adds (2 per pair, padding taps counted)."""
    n = case["n"]
    if case["kind"] == "dense":
        i, o = case["inputs"], case["outputs"]
        return {"bytes": 2 * (2 * n * i + 2 * n * o + i * o) + 4 * i * o + 8 * o, "flops": 3 * 2.0 * n * i * o}
    if case["kind"] == "vgg16":
        nbytes, flops = 0.0, 0.0
        for j, o in enumerate(_vgg16(case)):
            if o[0] == "conv":
                _, hw, c, k, pool = o
                weights, x, y, passes = 9 * c * k, n * hw * hw * c, n * hw * hw * k, 2 if j == 0 else 3
                flops += passes * 2.0 * n * hw * hw * k * 9 * c
            else:
                weights, x, y, passes = o[1] * o[2], n * o[1], n * o[2], 3
                flops += passes * 2.0 * n * o[1] * o[2]
            # x, weights and dy in; y, dx (but for the image) and the gradient out; the pool behind it: forward x in, y out, backward dy in, dx out
            nbytes += 6 * weights + (2 if j == 0 else 4) * x + 4 * y + (2 * 2.5 * y if o[0] == "conv" and o[4] else 0)
            nbytes += 20 * weights if case["update"] else 0      # momentum and weights in and out, the bf16 copy out
        return {"bytes": nbytes, "flops": flops}
    nbytes, flops = 0.0, 0.0
    e = 2 if case.get("dtype", BF16) == BF16 else 4
    for layer in _conv_layers(case):
        h, w, c, k, r, s = layer[:6]
        ho, wo = _out(layer)
        first = case["kind"] == "stem"
        nbytes += e * (n * h * w * c * (1 if first else 2) + 2 * n * ho * wo * k + k * r * s * c) + 4 * k * r * s * c + 4 * k
        flops += (2 if first else 3) * 2.0 * n * ho * wo * k * r * s * c
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case.get("dtype") == F32:
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 7e-3, "max": 1.6e-2}
