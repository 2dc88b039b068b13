"""The work that users of this library have it do, as measurable cases.

Every case is one pass through the public entry points: the layer calls
(`layer_forward` / `layer_backward`) on tensors in the library's layout, or
the PyTorch modules that `convert` puts into a model, on tensors in torch's
own layout.  Sizes are those of the repository's workloads (`synth/`,
`bench.py`) and of common networks; `draw` spreads them over the ranges they
come from, odd sizes and every mask included.  Both dtypes are here because
both are used: a torch model is float32 until its user says otherwise (the
paper's experiments are), bfloat16 is what large models train in.
"""
import math

import torch
import torch.nn.functional as F
from torch import nn

import paper_2404_12406_amd as ms
from paper_2404_12406_amd import autograd as msnn

# The ResNet-18-shaped stack trains its convolutions from this one on (its last
# stage).  Those have no ReLU behind them: where rounding turns a sign, a ReLU's
# gradient jumps, and two correct bfloat16 gradients would differ by far more
# than their rounding.
TRAINED = 13

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest call: one float32 3x3 convolution of a small network,
        # only its input gradient wanted.  Launches and host work are all of it.
        dict(name="conv_small_f32", kind="conv", dtype="f32", torch_layout=False, n=8, c=16, k=32, size="32x32",
             filter="3x3", stride=1, pad=1, mask=1),
        # The Linear layers of one transformer encoder layer on 16 x 512
        # tokens, weights frozen, gradients to the inputs: fine-tuning below an
        # adapter.  The repository's headline workload, one layer of it.
        dict(name="encoder_layer_bf16", kind="encoder", dtype="bf16", tokens=8192, hidden=768, ffn=3072),
        # A float32 fully connected layer, trained.
        dict(name="linear_train_f32", kind="linear", dtype="f32", m=4096, k=1024, n=4096, mask=7),
        # The convolution of the mask sweep (256 channels at 28 x 28), every flag.
        dict(name="conv_sweep_bf16", kind="conv", dtype="bf16", torch_layout=False, n=32, c=256, k=256, size="28x28",
             filter="3x3", stride=1, pad=1, mask=7),
        # A ResNet stage-1 convolution trained as a torch user has it: float32,
        # NCHW activations, through the module and autograd.
        dict(name="conv_train_f32", kind="conv", dtype="f32", torch_layout=True, n=32, c=64, k=64, size="56x56",
             filter="3x3", stride=1, pad=1, mask=7),
        # Channel counts and extents that no tile divides.
        dict(name="conv_ragged_bf16", kind="conv", dtype="bf16", torch_layout=False, n=16, c=60, k=100, size="57x45",
             filter="3x3", stride=2, pad=1, mask=7),
        # BN in evaluation mode with its scale and shift trained, behind the
        # first convolution of a ResNet.
        dict(name="bn_affine_bf16", kind="bn", dtype="bf16", n=64, c=64, size="112x112", mask=7),
        # The activations between an encoder layer's FFN Linears: ReLU with its
        # 1-bit mask, then dropout with its regenerated one, both ways.
        dict(name="relu_dropout_bf16", kind="activation", dtype="bf16", rows=8192, cols=3072, p=0.1),
        # A layer of a video network, every flag.
        dict(name="conv3d_bf16", kind="conv", dtype="bf16", torch_layout=False, n=8, c=64, k=64, size="16x56x56",
             filter="3x3x3", stride=1, pad=1, mask=7),
        # An upsampling layer of an image decoder, every flag.
        dict(name="conv_transpose_bf16", kind="conv_transpose", dtype="bf16", n=32, c=256, k=128, size="28x28",
             filter="4x4", stride=2, pad=1, mask=7),
        # The paper's synthetic deep CNN (8 channels, float32, 256 x 256
        # images, 3x3 convolutions without bias) with its later layers
        # differentiable, as a converted torch model.
        dict(name="synthetic_cnn_f32", kind="cnn", n=64, c=8, image=256, depth=6, first=3),
        # Transfer learning on a ResNet-18-shaped network: everything frozen
        # below the last stage, that stage's convolutions and the head trained.
        dict(name="resnet18_transfer_bf16", kind="resnet", n=64, image=224),
    ]


def _join(extents):
    return "x".join(str(e) for e in extents)


def _ints(extents):
    return [int(e) for e in extents.split("x")]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: usually what networks have, sometimes anything."""
    c = _log(rng, lo, hi)
    if rng.random() < 0.3:
        return c
    step = 8 if c < 64 else 32 if c < 256 else 64
    return max(step, (c + step // 2) // step * step)


def _mask(rng):
    return rng.choice([1, 1, 5, 6, 7, 7])


def _draw_conv(rng):
    dims = 3 if rng.random() < 0.2 else 2
    dtype = rng.choice(["f32", "bf16"])
    f = rng.choice([1, 3, 3, 3, 5]) if dims == 2 else rng.choice([1, 3])
    c, k = _channels(rng, 3, 512), _channels(rng, 8, 512)
    stride = rng.choice([1, 1, 1, 2])
    side = _log(rng, 7, 64) if dims == 2 else _log(rng, 7, 32)
    size = [side, max(1, side + rng.choice([0, 0, 0, -1, 3]))]
    if dims == 3:
        size = [_log(rng, 4, 16)] + size
    pixels = math.prod(size) / stride ** dims
    # at most the sweep layer's contraction (29.6 GFLOP) and 13M elements a tensor
    flops = 2 * pixels * c * k * f ** dims
    most = min(29.6e9 / flops, 13e6 / (math.prod(size) * c), 13e6 / (pixels * k))
    if most < 1:
        return _draw_conv(rng)
    return dict(kind="conv", dtype=dtype, torch_layout=dims == 2 and rng.random() < 0.4, n=_log(rng, 1, max(1, min(most, 64))), c=c,
                k=k, size=_join(size), filter=_join([f] * dims), stride=stride, pad=f // 2, mask=_mask(rng))


def _draw_linear(rng):
    m, k, n = _log(rng, 32, 8192), _channels(rng, 64, 4096), _channels(rng, 64, 4096)
    if m * k * n > 4096 * 1024 * 4096:
        m = 4096 * 1024 * 4096 // (k * n)
    return dict(kind="linear", dtype=rng.choice(["f32", "bf16"]), m=m, k=k, n=n, mask=_mask(rng))


def _draw_encoder(rng):
    hidden = 64 * rng.randint(4, 12)
    return dict(kind="encoder", dtype=rng.choice(["bf16", "bf16", "f32"]), tokens=_log(rng, 256, 4096), hidden=hidden,
                ffn=4 * hidden)


def _draw_bn(rng):
    c, side = _channels(rng, 16, 512), _log(rng, 7, 112)
    n = _log(rng, 1, max(1, min(64, 51e6 / (c * side * side))))
    return dict(kind="bn", dtype=rng.choice(["f32", "bf16"]), n=n, c=c, size=_join([side, side + rng.choice([0, 0, -1])]),
                mask=rng.choice([1, 6, 7]))


def _draw_activation(rng):
    rows = _log(rng, 64, 8192)
    return dict(kind="activation", dtype=rng.choice(["f32", "bf16"]), rows=rows, cols=_log(rng, 256, min(4096, 12e6 // rows)),
                p=rng.choice([0.1, 0.5]))


def _draw_conv_transpose(rng):
    c, k, side, f = _channels(rng, 16, 256), _channels(rng, 8, 128), _log(rng, 7, 28), rng.choice([2, 4, 4])
    return dict(kind="conv_transpose", dtype=rng.choice(["f32", "bf16"]), n=_log(rng, 1, 16), c=c, k=k, size=_join([side, side]),
                filter=_join([f, f]), stride=2, pad=f // 2 - 1, mask=_mask(rng))


def _draw_cnn(rng):
    depth = rng.randint(2, 6)
    return dict(kind="cnn", n=_log(rng, 1, 32), c=rng.choice([3, 8, 8, 16]), image=_log(rng, 32, 224), depth=depth,
                first=rng.randint(0, depth - 1))


def _draw_resnet(rng):
    return dict(kind="resnet", n=_log(rng, 1, 32), image=32 * rng.randint(2, 7))


def draw(rng):
    return rng.choice([_draw_conv, _draw_conv, _draw_conv, _draw_linear, _draw_linear, _draw_encoder, _draw_bn,
                       _draw_activation, _draw_conv_transpose, _draw_cnn, _draw_resnet])(rng)


# ------------------------------------------------------------------ inputs
class _Maker:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, dtype, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.g, device="cuda") * std + mean).to(dtype)

    def uniform(self, shape, dtype, lo, hi):
        return (torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo).to(dtype)

    def kaiming(self, shape, dtype, fan_in):
        r = 1.0 / math.sqrt(fan_in)
        return self.uniform(shape, dtype, -r, r)


def _cl(t):
    return t.contiguous(memory_format=torch.channels_last if t.dim() == 4 else torch.channels_last_3d)


def _out_size(case):
    if case["kind"] == "conv":
        return [(s + 2 * case["pad"] - f) // case["stride"] + 1 for s, f in zip(_ints(case["size"]), _ints(case["filter"]))]
    return [(s - 1) * case["stride"] - 2 * case["pad"] + f for s, f in zip(_ints(case["size"]), _ints(case["filter"]))]


def _stages(case):
    """(in, out, stride) of the 3x3 convolutions of the ResNet-18-shaped stack."""
    out, c = [], 64
    for k in (64, 128, 256, 512):
        for j in range(4):
            out.append((c, k, 2 if j == 0 else 1))
            c = k
    return out


def _layer_inputs(case, mk):
    """x, W, b, dy of a single conv, transposed conv or linear case, in torch's layout."""
    dt = DTYPES[case["dtype"]]
    if case["kind"] == "linear":
        x, w = (case["m"], case["k"]), (case["n"], case["k"])
        fan, nb, y = case["k"], case["n"], (case["m"], case["n"])
    else:
        x = (case["n"], case["c"], *_ints(case["size"]))
        y = (case["n"], case["k"], *_out_size(case))
        f = tuple(_ints(case["filter"]))
        w = (case["k"], case["c"]) + f if case["kind"] == "conv" else (case["c"], case["k"]) + f
        fan, nb = w[1] * math.prod(f), case["k"]
    return mk.normal(x, dt), mk.kaiming(w, dt, fan), mk.kaiming((nb,), dt, fan), mk.normal(y, dt)


def _encoder_layers(case, mk):
    """(x or None when it is the previous layer's output, W, b, dy or None when
    it is the next layer's input gradient) of QKV, out, FFN up and FFN down."""
    dt, t, h, f = DTYPES[case["dtype"]], case["tokens"], case["hidden"], case["ffn"]
    out = []
    for kin, n, own_x, own_dy in ((h, 3 * h, True, True), (h, h, True, True), (h, f, True, False), (f, h, False, True)):
        out.append((mk.normal((t, kin), dt) if own_x else None, mk.normal((n, kin), dt, 0.02), mk.normal((n,), dt, 0.02),
                    mk.normal((t, n), dt) if own_dy else None))
    return out


def _bn_inputs(case, mk):
    dt, c = DTYPES[case["dtype"]], case["c"]
    shape = (case["n"], c, *_ints(case["size"]))
    return (mk.normal(shape, dt), mk.uniform((c,), dt, 0.5, 1.5), mk.normal((c,), dt, 0.1), mk.normal((c,), dt, 0.1),
            mk.uniform((c,), dt, 0.5, 1.5), mk.normal(shape, dt))


def _cnn_inputs(case, mk):
    c, f32 = case["c"], torch.float32
    ws = [mk.kaiming((c, c, 3, 3), f32, 9 * c) for _ in range(case["depth"])]
    shape = (case["n"], c, case["image"], case["image"])
    return mk.normal(shape, f32), ws, mk.normal(shape, f32)


def _resnet_inputs(case, mk):
    """Image, [(W, stride, mean, var, gamma, beta)] of stem and stages, head W
    and b, logit gradients.  Filters have the variance that keeps activations
    at one scale, with a ReLU behind the convolution or without."""
    dt = torch.bfloat16
    convs = []
    for i, (c, k, stride, r) in enumerate([(3, 64, 2, 7)] + [(c, k, s, 3) for c, k, s in _stages(case)]):
        w = mk.normal((k, c, r, r), dt, math.sqrt((2.0 if i < TRAINED else 1.0) / (c * r * r)))
        convs.append((w, stride, mk.normal((k,), dt, 0.1), mk.uniform((k,), dt, 0.5, 1.5), mk.uniform((k,), dt, 0.5, 1.5),
                      mk.normal((k,), dt, 0.1)))
    x = mk.normal((case["n"], 3, case["image"], case["image"]), dt)
    return x, convs, mk.kaiming((1000, 512), dt, 512), mk.kaiming((1000,), dt, 512), mk.normal((case["n"], 1000), dt)


def prepare(case, seed):
    mk = _Maker(seed)
    kind, st = case["kind"], {"case": case}
    if kind in ("conv", "conv_transpose", "linear"):
        x, w, b, dy = _layer_inputs(case, mk)
        mask = case["mask"]
        if kind == "linear":
            st.update(spec=ms.Linear(), x=x, w=w, b=b, dy=dy)
        elif case.get("torch_layout"):
            layer = nn.Conv2d(case["c"], case["k"], _ints(case["filter"])[0], case["stride"], case["pad"], device="cuda", dtype=x.dtype)
            with torch.no_grad():
                layer.weight.copy_(w)
                layer.bias.copy_(b)
            layer.weight.requires_grad_(bool(mask & 2))
            layer.bias.requires_grad_(bool(mask & 4))
            x.requires_grad_(bool(mask & 1))
            model = msnn.convert(nn.Sequential(layer))
            st.update(model=model, x=x, dy=dy, wrt=[t for t in (x, *model.parameters()) if t.requires_grad])
        else:
            if kind == "conv_transpose":
                spec = ms.ConvTranspose2d(case["stride"], case["pad"])
            else:
                spec = (ms.Conv2d if len(_ints(case["size"])) == 2 else ms.Conv3d)(case["stride"], case["pad"])
            st.update(spec=spec, x=_cl(x), w=_cl(w), b=b, dy=_cl(dy))
    elif kind == "encoder":
        st.update(layers=_encoder_layers(case, mk))
    elif kind == "bn":
        x, gamma, beta, mean, var, dy = _bn_inputs(case, mk)
        st.update(spec=ms.BatchNormEval(mean, var), x=_cl(x), w=gamma, b=beta, dy=_cl(dy))
    elif kind == "activation":
        shape, dt = (case["rows"], case["cols"]), DTYPES[case["dtype"]]
        st.update(x=mk.normal(shape, dt), dy=mk.normal(shape, dt), key=seed)
    elif kind == "cnn":
        x, ws, dy = _cnn_inputs(case, mk)
        c = case["c"]
        model = nn.Sequential(*[nn.Conv2d(c, c, 3, padding=1, bias=False, device="cuda") for _ in ws])
        with torch.no_grad():
            for i, w in enumerate(ws):
                model[i].weight.copy_(w)
                model[i].weight.requires_grad_(i >= case["first"])
        model = msnn.convert(model)
        st.update(model=model, x=x, dy=dy, wrt=[p for p in model.parameters() if p.requires_grad])
    elif kind == "resnet":
        x, convs, hw, hb, dy = _resnet_inputs(case, mk)
        layers = []
        for w, stride, mean, var, gamma, beta in convs:
            conv = nn.Conv2d(w.shape[1], w.shape[0], w.shape[2], stride, w.shape[2] // 2, bias=False, device="cuda", dtype=w.dtype)
            bn = nn.BatchNorm2d(w.shape[0], device="cuda", dtype=w.dtype).eval()
            with torch.no_grad():
                for dst, src in ((conv.weight, w), (bn.running_mean, mean), (bn.running_var, var), (bn.weight, gamma),
                                 (bn.bias, beta)):
                    dst.copy_(src)
            layers += [conv, bn, nn.ReLU()] if len(layers) < 3 * TRAINED else [conv, bn]
        head = nn.Linear(512, 1000, device="cuda", dtype=x.dtype)
        with torch.no_grad():
            head.weight.copy_(hw)
            head.bias.copy_(hb)
        model = msnn.convert(nn.Sequential(*layers, nn.AdaptiveAvgPool2d(1), nn.Flatten(), head))
        trained = [m for m in model if isinstance(m, msnn.MSConv2d)][-4:] + [m for m in model if isinstance(m, msnn.MSLinear)]
        for p in model.parameters():
            p.requires_grad_(False)
        for m in trained:
            m.requires_grad_(True)
        st.update(model=model, x=x, dy=dy, wrt=[p for p in model.parameters() if p.requires_grad])
    else:
        raise ValueError(kind)
    return st


def run(st):
    case = st["case"]
    if "model" in st:
        y = st["model"](st["x"])
        return (y.detach(), *torch.autograd.grad(y, st["wrt"], st["dy"]))
    if case["kind"] == "encoder":
        outs, recs, y = [], [], None
        for x, w, b, _ in st["layers"]:
            y, rec = ms.layer_forward(ms.Linear(), y if x is None else x, w, b, ms.MASK_INPUT)
            outs.append(y)
            recs.append(rec)
        gx = None
        for (_, _, _, dy), rec in zip(reversed(st["layers"]), reversed(recs)):
            gx = ms.layer_backward(rec, gx if dy is None else dy)[0]
            outs.append(gx)
        return outs
    if case["kind"] == "activation":
        h, r1 = ms.layer_forward(ms.ReLU(), st["x"], mask=ms.MASK_INPUT)
        y, r2 = ms.layer_forward(ms.Dropout(case["p"], st["key"], 0), h, mask=ms.MASK_INPUT)
        gh = ms.layer_backward(r2, st["dy"])[0]
        return h, y, gh, ms.layer_backward(r1, gh)[0]
    y, rec = ms.layer_forward(st["spec"], st["x"], st["w"], st["b"], case["mask"])
    return (y, *[g for g in ms.layer_backward(rec, st["dy"]) if g is not None])


# ------------------------------------------------------------------ what a pass cannot do without
def _elt(case):
    return 4 if case.get("dtype", "f32") == "f32" else 2


def _contraction(mask, macs, nx, nw, nb, ny, elt):
    """Work of one masked linear layer call, forward and backward: every
    operand of each direction read once, every result written once."""
    passes = 1 + (mask & 1) + (mask >> 1 & 1)
    moved = nx + nw + nb + ny
    if mask:
        moved += ny
    if mask & 1:
        moved += nw + nx
    if mask & 2:
        moved += nx + nw
    if mask & 4:
        moved += nb
    return moved * elt, 2 * macs * passes


def work(case):
    kind = case["kind"]
    if kind in ("conv", "conv_transpose"):
        f, cin, cout = math.prod(_ints(case["filter"])), case["c"], case["k"]
        xin, yout = math.prod(_ints(case["size"])), math.prod(_out_size(case))
        macs = case["n"] * (yout if kind == "conv" else xin) * cin * cout * f
        b, fl = _contraction(case["mask"], macs, case["n"] * cin * xin, cin * cout * f, cout, case["n"] * cout * yout, _elt(case))
    elif kind == "linear":
        m, k, n = case["m"], case["k"], case["n"]
        b, fl = _contraction(case["mask"], m * k * n, m * k, k * n, n, m * n, _elt(case))
    elif kind == "encoder":
        t, h, f = case["tokens"], case["hidden"], case["ffn"]
        b = fl = 0
        for kin, n in ((h, 3 * h), (h, h), (h, f), (f, h)):
            bi, fi = _contraction(1, t * kin * n, t * kin, kin * n, n, t * n, _elt(case))
            b, fl = b + bi, fl + fi
    elif kind == "bn":
        n = case["n"] * case["c"] * math.prod(_ints(case["size"]))
        m = case["mask"]
        b, fl = n * _elt(case) * (2 + 1 + (m & 1) + (m >> 1 & 1)), 8 * n
    elif kind == "activation":
        n = case["rows"] * case["cols"]
        b, fl = 8 * n * _elt(case) + n // 4, 4 * n   # four passes, and the bits written and read
    elif kind == "cnn":
        # layer by layer: each is an autograd node whose output autograd holds
        c, n, px, b, fl = case["c"], case["n"], case["image"] ** 2, 0, 0
        for i in range(case["depth"]):
            mask = (1 if i > case["first"] else 0) | (2 if i >= case["first"] else 0)
            bi, fi = _contraction(mask, n * px * c * c * 9, n * px * c, 9 * c * c, 0, n * px * c, 4)
            b, fl = b + bi, fl + fi
    else:
        n, side, b, fl = case["n"], case["image"], 0, 0
        convs = [(3, 64, 2, 7)] + [(c, k, s, 3) for c, k, s in _stages(case)]
        for i, (c, k, s, r) in enumerate(convs):
            out = (side + 2 * (r // 2) - r) // s + 1
            mask = (1 if i > TRAINED else 0) | (2 if i >= TRAINED else 0)
            ny = n * k * out * out
            bi, fi = _contraction(mask, ny * c * r * r, n * c * side * side, k * c * r * r, 0, ny, 2)
            # behind it BN and a ReLU, or BN both ways: two passes, each read and written
            b, fl, side = b + bi + 2 * 2 * 2 * ny, fl + fi + 4 * ny, out
        bi, fi = _contraction(7, n * 512 * 1000, n * 512, 512 * 1000, 1000, n * 1000, 2)
        b, fl = b + bi, fl + fi
    return {"bytes": b, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind == "activation":
        return "exact"   # a select, a product rounded once, and a fixed generator
    if kind == "resnet":
        # bf16 activations through 17 convolutions and norms
        return {"rel": 0.03, "max": 0.6}
    if kind == "cnn" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 5e-5}
    # one rounding to bf16 (2^-9) from sums in 32 bits; the encoder's chained
    # layers round twice
    return {"rel": 8e-3, "max": 4e-2}


# ------------------------------------------------------------------ the same in 64 bits
def _conv(x, w, stride, pad):
    """Cross-correlation in any number of dimensions, tap by tap as matrix
    products, from torch operations that differentiate."""
    dims = x.dim() - 2
    x = F.pad(x, [pad] * (2 * dims)).movedim(1, -1)
    taps = w.shape[2:]
    out = [(x.shape[1 + d] - taps[d]) // stride + 1 for d in range(dims)]
    y = 0
    for tap in torch.cartesian_prod(*[torch.arange(t) for t in taps]).reshape(-1, dims).tolist():
        sl = tuple(slice(t, t + (o - 1) * stride + 1, stride) for t, o in zip(tap, out))
        y = y + x[(slice(None), *sl)] @ w[(slice(None), slice(None), *tap)].t()
    return y.movedim(-1, 1)


def _conv_transpose(x, w, stride, pad, out):
    y = x.new_zeros((x.shape[0], w.shape[1], *[o + 2 * pad for o in out]))
    xm = x.movedim(1, -1)
    for tap in torch.cartesian_prod(*[torch.arange(t) for t in w.shape[2:]]).reshape(-1, len(out)).tolist():
        sl = tuple(slice(t, t + (s - 1) * stride + 1, stride) for t, s in zip(tap, x.shape[2:]))
        part = (xm @ w[(slice(None), slice(None), *tap)]).movedim(-1, 1)
        full = torch.zeros_like(y)
        full[(slice(None), slice(None), *sl)] = part
        y = y + full
    return y[(slice(None), slice(None), *[slice(pad, pad + o) for o in out])]


def _per_channel(t, like):
    return t.view(1, -1, *[1] * (like.dim() - 2))


def _bn(x, mean, var, gamma, beta, eps=1e-5):
    s = gamma / torch.sqrt(var + eps)
    return x * _per_channel(s, x) + _per_channel(beta - mean * s, x)


def exact(case, seed):
    mk, kind = _Maker(seed), case["kind"]

    def wide(*ts):
        return [t.double() for t in ts]

    if kind == "activation":
        # which elements a dropout keeps is the library's generator's affair
        shape, dt = (case["rows"], case["cols"]), DTYPES[case["dtype"]]
        return mk.normal(shape, dt).double().clamp(min=0), None, None, None
    if kind == "encoder":
        outs, y, layers = [], None, _encoder_layers(case, mk)
        for x, w, b, _ in layers:
            x, w, b = wide(x if x is not None else y, w, b)
            y = x @ w.t() + b
            outs.append(y)
        gx = None
        for _, w, _, dy in reversed(layers):
            gx = (gx if dy is None else dy.double()) @ w.double()
            outs.append(gx)
        return outs
    if kind == "cnn":
        x, ws, dy = _cnn_inputs(case, mk)
        ws = [w.double().requires_grad_(i >= case["first"]) for i, w in enumerate(ws)]
        y = x.double()
        for w in ws:
            y = _conv(y, w, 1, 1)
        return (y.detach(), *torch.autograd.grad(y, ws[case["first"]:], dy.double()))
    if kind == "resnet":
        x, convs, hw, hb, dy = _resnet_inputs(case, mk)
        y, ws = x.double(), []
        for i, (w, stride, *stats) in enumerate(convs):
            w = w.double().requires_grad_(i >= TRAINED)
            if i >= TRAINED:
                ws.append(w)
            mean, var, gamma, beta = wide(*stats)
            y = _bn(_conv(y, w, stride, w.shape[2] // 2), mean, var, gamma, beta)
            y = y.clamp(min=0) if i < TRAINED else y
        hw, hb = [t.requires_grad_(True) for t in wide(hw, hb)]
        y = y.mean(dim=(2, 3)) @ hw.t() + hb
        return (y.detach(), *torch.autograd.grad(y, [*ws, hw, hb], dy.double()))
    if kind == "bn":
        x, gamma, beta, mean, var, dy = wide(*_bn_inputs(case, mk))
        x, w, b = [t.requires_grad_(True) for t in (x, gamma, beta)]
        y = _bn(x, mean, var, w, b)
    else:
        x, w, b, dy = wide(*_layer_inputs(case, mk))
        x, w, b = [t.requires_grad_(True) for t in (x, w, b)]
        if kind == "linear":
            y = x @ w.t() + b
        elif kind == "conv":
            y = _conv(x, w, case["stride"], case["pad"])
            y = y + _per_channel(b, y)
        else:
            y = _conv_transpose(x, w, case["stride"], case["pad"], _out_size(case))
            y = y + _per_channel(b, y)
    wrt = [t for bit, t in ((1, x), (2, w), (4, b)) if case["mask"] & bit]
    return (y.detach(), *torch.autograd.grad(y, wrt, dy))
