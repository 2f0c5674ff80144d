"""Performance cases of the fused-block executor: operator graphs of this repository's workload shapes, planned and run
through the library's public calls (`api.Graph`, `Graph.rewrite`, `api.Plan`, `Plan.prepare`, `Plan.run`).

A case names a kind of graph, its sizes, the storage type and the plan options.  `prepare` builds the graph, puts
seeded weights and inputs on the GPU and builds the plan, as a serving program does once; `run` is one inference.

Plan options.  A program that serves one fixed shape for long tunes its plan on the device (`tuned`); one that meets a
shape now and then takes the generator's own choice of tiles, the default of `api.Session`.  `layout`, `attention` and
`extensions` (broadcast prologue and squeeze-excite tails) are the documented plan options of the same names.
"""
import math

import numpy as np
import torch

from paper_2108_13342_amd import api
from paper_2108_13342_amd.build import CACHE

TORCH_TYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i64": torch.int64, "bool": torch.bool}
TYPE_BYTES = {"f32": 4, "f16": 2, "bf16": 2, "i64": 8, "bool": 1}
CAST_CODE = {"f32": 1, "f16": 10, "bf16": 16, "i64": 7, "bool": 9}
PROFILE_BYTES = 2 << 30      # device memory the plan builder may time candidates in (tuned plans only)

# (expand, kernel, out channels, repeats, first stride)
EFFNET_B0_STAGES = [(1, 3, 16, 1, 1), (6, 3, 24, 2, 2), (6, 5, 40, 2, 2), (6, 3, 80, 3, 2),
                    (6, 5, 112, 3, 1), (6, 5, 192, 4, 2), (6, 3, 320, 1, 1)]


# ------------------------------------------------------------------------------------------------ graph recording
class _Net:
    """Records tensors and operators; `fill` of an input or weight makes its values from a torch.Generator."""

    def __init__(self, dtype):
        self.dtype = dtype
        self.tensors = {}        # name -> [dtype, shape, kind, fill, host value of a scalar constant]
        self.ops = []
        self.flops = 0.0

    def _add(self, name, dtype, shape, kind, fill=None, value=None):
        self.tensors[name] = [dtype, tuple(int(d) for d in shape), kind, fill, value]
        return name

    def input(self, name, shape, fill, dtype=None):
        return self._add(name, dtype or self.dtype, shape, "input", fill)

    def weight(self, name, shape, fill, dtype=None):
        return self._add(name, dtype or self.dtype, shape, "weight", fill)

    def const(self, name, value, dtype=None):
        value = float(torch.tensor(value).to(TORCH_TYPES[dtype or self.dtype]))      # the compiler is told what is stored
        return self._add(name, dtype or self.dtype, (), "weight", lambda gen, shape: torch.full(shape, value), value)

    def shape(self, name):
        return self.tensors[name][1]

    def op(self, kind, inputs, shape, attrs=None, dtype=None, name=None):
        shapes = shape if isinstance(shape, list) else [shape]
        outs = [self._add(name or f"t{len(self.tensors)}", dtype or self.dtype, s, "intermediate") for s in shapes]
        self.ops.append((kind, list(inputs), outs, dict(attrs or {})))
        return outs if isinstance(shape, list) else outs[0]

    def output(self, name):
        self.tensors[name][2] = "output"

    # -- the operators the graphs below are made of
    def ew(self, kind, *inputs, attrs=None):
        return self.op(kind, inputs, torch.broadcast_shapes(*[self.shape(i) for i in inputs]), attrs)

    def matmul(self, x, w, share=1.0):
        """share: the part of the products that the result depends on (a causal mask drops the others)."""
        sx, sw = self.shape(x), self.shape(w)
        out = tuple(torch.broadcast_shapes(sx[:-2], sw[:-2])) + (sx[-2], sw[-1])
        self.flops += 2.0 * math.prod(out) * sx[-1] * share
        return self.op("MatMul", [x, w], out)

    def conv(self, x, w, bias, stride, pad, group=1):
        n, _, h, wd = self.shape(x)
        co, cig, kh, kw = self.shape(w)
        out = (n, co, (h + 2 * pad - kh) // stride + 1, (wd + 2 * pad - kw) // stride + 1)
        self.flops += 2.0 * math.prod(out) * cig * kh * kw
        return self.op("Conv", [x, w] + ([bias] if bias else []), out, {"strides": [stride] * 2, "pads": [pad] * 4, "group": group})

    def reshape(self, x, shape):
        return self.op("Reshape", [x], shape, {"shape": [int(d) for d in shape]}, self.tensors[x][0])

    def transpose(self, x, perm):
        s = self.shape(x)
        return self.op("Transpose", [x], tuple(s[p] for p in perm), {"perm": list(perm)})

    def unsqueeze(self, x, axis):
        s = list(self.shape(x))
        s.insert(axis, 1)
        return self.op("Unsqueeze", [x], tuple(s), {"axes": [axis], "out_shape": s}, self.tensors[x][0])

    def reduce(self, kind, x):
        return self.op(kind, [x], self.shape(x)[:-1] + (1,), {"axes": [len(self.shape(x)) - 1], "keepdims": 1})

    def cast(self, x, to):
        return self.op("Cast", [x], self.shape(x), {"to": CAST_CODE[to]}, to)

    def bytes(self):
        """Every input and weight read once, every output written once."""
        return float(sum(TYPE_BYTES[t[0]] * math.prod(t[1]) for t in self.tensors.values() if t[2] != "intermediate"))


def _normal(mean=0.0, std=1.0):
    return lambda gen, shape: torch.randn(shape, generator=gen, device=gen.device) * std + mean


def _uniform(lo, hi):
    return lambda gen, shape: torch.rand(shape, generator=gen, device=gen.device) * (hi - lo) + lo


# ------------------------------------------------------------------------------------------------ the graphs
def residual_block(c):
    """3x3 convolution -> BatchNormalization -> Relu -> Add identity -> Relu."""
    n, ch, h, w = c["N"], c["C"], c["H"], c["W"]
    b = _Net(c["dtype"])
    x = b.input("x", (n, ch, h, w), _normal())
    cw = b.weight("conv_w", (ch, ch, 3, 3), _normal(0.0, math.sqrt(2.0 / (ch * 9))))
    bn = [b.weight(k, (ch,), f) for k, f in (("gamma", _uniform(0.5, 1.5)), ("beta", _normal(0.0, 0.1)), ("mean", _normal(0.0, 0.1)), ("var", _uniform(0.5, 1.5)))]
    y = b.conv(x, cw, None, 1, 1)
    y = b.op("BatchNormalization", [y] + bn, b.shape(y), {"epsilon": 1e-5})
    y = b.ew("Relu", y)
    b.output(b.ew("Relu", b.ew("Add", y, x)))
    return b


def resnet_stage(c):
    """Stem convolution, a basic block, a strided convolution that doubles the channels, a basic block."""
    b = _Net(c["dtype"])
    t = b.input("x", (c["N"], 3, c["R"], c["R"]), _normal())

    def conv(t, cout, stride=1):
        cin, k = b.shape(t)[1], len(b.ops)
        w = b.weight(f"w{k}", (cout, cin, 3, 3), _normal(0.0, math.sqrt(1.0 / (cin * 9))))
        return b.conv(t, w, b.weight(f"b{k}", (cout,), _normal(0.0, 0.1)), stride, 1)

    def basic(t):
        y = conv(b.ew("Relu", conv(t, b.shape(t)[1])), b.shape(t)[1])
        return b.ew("Relu", b.ew("Add", y, t))

    t = basic(b.ew("Relu", conv(t, c["C"])))
    b.output(basic(b.ew("Relu", conv(t, 2 * c["C"], 2))))
    return b


def memory_bound_chain(c):
    """rounds x 8 One-to-One layers (15 operators), then NCHW -> NHWC, reshape and channel shuffle."""
    n, ch, h, w, groups = c["N"], c["C"], c["H"], c["W"], c["groups"]
    b = _Net(c["dtype"])
    y = b.input("x", (n, ch, h, w), _normal())
    for r in range(c["rounds"]):
        for kind, k in (("Add", "c1"), ("Mul", "c2")):
            y = b.ew(kind, y, b.weight(f"r{r}_{k}", (1, ch, 1, 1), _uniform(-1.0, 1.0)))
        y = b.ew("Clip", y, attrs={"min": -4.0, "max": 4.0})
        for kind in ("Exp", "Sigmoid", "Tanh"):
            y = b.ew(kind, y)
        y = _gelu_erf(b, y, f"r{r}_gelu")
        y = b.ew("Pow", y, b.const(f"r{r}_two", 2.0))
        y = b.ew("Abs", y)
        y = b.ew("Add", y, b.const(f"r{r}_one", 1.0))
        y = b.ew("Sqrt", y)
    y = b.reshape(b.transpose(y, (0, 2, 3, 1)), (n, h * w, ch))
    y = b.transpose(b.reshape(y, (n, h * w, groups, ch // groups)), (0, 1, 3, 2))
    b.output(b.reshape(y, (n, h * w, ch)))
    return b


def _gelu_erf(b, x, tag):
    r2, one, half = b.const(f"{tag}_sqrt2", math.sqrt(2.0)), b.const(f"{tag}_one", 1.0), b.const(f"{tag}_half", 0.5)
    t = b.ew("Add", b.ew("Erf", b.ew("Div", x, r2)), one)
    return b.ew("Mul", b.ew("Mul", x, t), half)


def _gelu_tanh(b, x, tag):
    """The tanh form; Pow sits between Casts in a 16-bit graph."""
    three, c0, c1 = b.const(f"{tag}_three", 3.0), b.const(f"{tag}_c0", 0.044715), b.const(f"{tag}_c1", math.sqrt(2.0 / math.pi))
    one, half = b.const(f"{tag}_one", 1.0), b.const(f"{tag}_half", 0.5)
    if b.dtype != "f32":
        t = b.cast(x, "f32")
        t = b.op("Pow", [t, b.cast(three, "f32")], b.shape(x), dtype="f32")
        t = b.cast(t, b.dtype)
    else:
        t = b.ew("Pow", x, three)
    t = b.ew("Mul", b.ew("Add", x, b.ew("Mul", t, c0)), c1)
    t = b.ew("Add", b.ew("Tanh", t), one)
    return b.ew("Mul", b.ew("Mul", x, t), half)


def _layernorm(b, x, width, tag, in_f32=False):
    """The usual nine operators; in_f32: between Casts, as a 16-bit export of the decoder keeps it."""
    keep = b.dtype
    gamma = b.weight(f"{tag}_gamma", (width,), _normal(1.0, 0.02))
    beta = b.weight(f"{tag}_beta", (width,), _normal(0.0, 0.02))
    two = b.const(f"{tag}_two", 2.0)
    in_f32 = in_f32 and keep != "f32"
    if in_f32:
        x = b.cast(x, "f32")
        b.dtype = "f32"
    eps = b.const(f"{tag}_eps", 1e-5)
    d = b.ew("Sub", x, b.reduce("ReduceMean", x))
    if in_f32:
        two = b.cast(two, "f32")
    var = b.reduce("ReduceMean", b.ew("Pow", d, two))
    y = b.ew("Add", b.ew("Mul", b.ew("Div", d, b.ew("Sqrt", b.ew("Add", var, eps))), gamma), beta)
    b.dtype = keep
    return b.cast(y, keep) if in_f32 else y


def encoder_layer(c):
    """Post-LayerNorm encoder layer with an additive padding mask over the last tenth of the keys."""
    B, S, D, NH, F = c["B"], c["S"], c["D"], c["NH"], c["F"]
    b = _Net(c["dtype"])
    hd = D // NH
    x = b.input("x", (B, S, D), _normal())

    def padding(gen, shape):
        m = torch.zeros(shape, device=gen.device)
        m[..., S - S // 10:] = -1e4
        return m

    mask = b.weight("attn_mask", (B, 1, 1, S), padding)

    def lin(name, inp, k, n):
        w, bias = b.weight(f"{name}_w", (k, n), _normal(0.0, 0.02)), b.weight(f"{name}_b", (n,), _normal(0.0, 0.02))
        return b.ew("Add", b.matmul(inp, w), bias)

    q, k, v = b.op("Split", [lin("qkv", x, D, 3 * D)], [(B, S, D)] * 3, {"axis": 2, "split": [D, D, D]})
    q = b.transpose(b.reshape(q, (B, S, NH, hd)), (0, 2, 1, 3))
    k = b.transpose(b.reshape(k, (B, S, NH, hd)), (0, 2, 3, 1))
    v = b.transpose(b.reshape(v, (B, S, NH, hd)), (0, 2, 1, 3))
    s = b.ew("Mul", b.matmul(q, k), b.const("attn_scale", 1.0 / math.sqrt(hd)))
    s = b.ew("Add", s, mask)
    p = b.op("Softmax", [s], b.shape(s), {"axis": -1})
    o = b.reshape(b.transpose(b.matmul(p, v), (0, 2, 1, 3)), (B, S, D))
    h = _layernorm(b, b.ew("Add", lin("attn_out", o, D, D), x), D, "ln1")
    f = lin("ffn2", _gelu_erf(b, lin("ffn1", h, D, F), "ffn_gelu"), F, D)
    b.output(_layernorm(b, b.ew("Add", f, h), D, "ln2"))
    return b


def efficientnet(c):
    """Stem and the first `stages` stages of MBConv blocks with squeeze-excite, BatchNorm folded."""
    b = _Net(c["dtype"])
    y = b.input("x", (c["N"], 3, c["R"], c["R"]), _normal())

    def conv(name, inp, cout, k, stride, group=1):
        fan = b.shape(inp)[1] // group * k * k
        w = b.weight(f"{name}_w", (cout, b.shape(inp)[1] // group, k, k), _normal(0.0, math.sqrt(2.0 / fan)))
        return b.conv(inp, w, b.weight(f"{name}_b", (cout,), _normal(0.0, 0.1)), stride, k // 2, group)

    def swish(x):
        return b.ew("Mul", x, b.ew("Sigmoid", x))

    y = swish(conv("stem", y, 32, 3, 2))
    bi = 0
    for e, k, cout, reps, s0 in EFFNET_B0_STAGES[:c["stages"]]:
        for r in range(reps):
            bi += 1
            cin, stride, t = b.shape(y)[1], s0 if r == 0 else 1, y
            if e != 1:
                t = swish(conv(f"mb{bi}_expand", t, cin * e, 1, 1))
            n, ch = b.shape(t)[:2]
            t = swish(conv(f"mb{bi}_dw", t, ch, k, stride, group=ch))
            sq = b.op("GlobalAveragePool", [t], (n, ch, 1, 1))
            sq = swish(conv(f"mb{bi}_se1", sq, max(1, cin // 4), 1, 1))
            sq = b.ew("Sigmoid", conv(f"mb{bi}_se2", sq, ch, 1, 1))
            t = conv(f"mb{bi}_project", b.ew("Mul", t, sq), cout, 1, 1)
            y = b.ew("Add", t, y) if stride == 1 and cin == cout else t
    b.output(y)
    return b


def decoder(c):
    """Pre-LayerNorm causal decoder stack with a tied vocabulary projection, at an exporter's granularity; returns every
    layer's stacked key / value beside the logits."""
    B, S, D, NH, F, L, V, P = c["B"], c["S"], c["D"], c["NH"], 4 * c["D"], c["L"], c["V"], max(1024, c["S"])
    b = _Net(c["dtype"])
    dt, hd = c["dtype"], D // NH
    causal = (S + 1) / (2.0 * S)
    ids = b.input("input_ids", (B, S), lambda gen, shape: torch.randint(0, V, shape, generator=gen, device=gen.device), "i64")

    def real_tokens(gen, shape):      # sequences of unequal length, padded on the right
        length = torch.randint((S + 1) // 2, S + 1, (B, 1), generator=gen, device=gen.device)
        return torch.arange(S, device=gen.device).expand(B, S) < length

    amask = b.input("attention_mask", (B, S), real_tokens, "i64")
    wte = b.weight("wte", (V, D), _normal(0.0, 0.02))
    wpe = b.weight("wpe", (P, D), _normal(0.0, 0.02))
    maskbuf = b.weight("causal_bias", (1, 1, P, P), lambda gen, shape: torch.tril(torch.ones(shape, dtype=torch.bool, device=gen.device)), "bool")
    pos_ids = b._add("position_ids", "i64", (1, S), "weight", lambda gen, shape: torch.arange(S, device=gen.device).reshape(shape), np.arange(S))
    mask_value = b.const("mask_value", -1e4)

    def lin(name, inp, k, n):
        w, bias = b.weight(f"{name}_w", (k, n), _normal(0.0, 0.02)), b.weight(f"{name}_b", (n,), _normal(0.0, 0.02))
        lead = b.shape(inp)[:-1]
        return b.reshape(b.ew("Add", b.matmul(b.reshape(inp, (math.prod(lead), k)), w), bias), tuple(lead) + (n,))

    tok = b.op("Gather", [wte, b.reshape(ids, (B, S))], (B, S, D), {"axis": 0})
    h = b.ew("Add", tok, b.op("Gather", [wpe, pos_ids], (1, S, D), {"axis": 0}))
    em = b.cast(b.unsqueeze(b.unsqueeze(amask, 1), 2), dt)
    em = b.ew("Mul", b.ew("Sub", b.const("pad_one", 1.0), em), b.const("pad_value", -1e4))
    for l in range(L):
        a = _layernorm(b, h, D, f"l{l}_ln1", True)
        q, k, v = b.op("Split", [lin(f"l{l}_attn", a, D, 3 * D)], [(B, S, D)] * 3, {"axis": 2, "split": [D, D, D]})
        q = b.transpose(b.reshape(q, (B, S, NH, hd)), (0, 2, 1, 3))
        k = b.transpose(b.reshape(k, (B, S, NH, hd)), (0, 2, 3, 1))
        v = b.transpose(b.reshape(v, (B, S, NH, hd)), (0, 2, 1, 3))
        b.output(b.op("Concat", [b.unsqueeze(b.transpose(k, (0, 1, 3, 2)), 0), b.unsqueeze(v, 0)], (2, B, NH, S, hd), {"axis": 0}, name=f"present_{l}"))
        s = b.matmul(q, k, causal)
        hd_c = b._add(f"l{l}_head_size", "i64", (), "weight", lambda gen, shape: torch.full(shape, hd), hd)
        s = b.ew("Div", s, b.ew("Sqrt", b.cast(hd_c, dt)))
        m = b.op("Slice", [maskbuf], (1, 1, S, P), {"starts": [0], "ends": [S], "axes": [2]}, "bool")
        m = b.op("Slice", [m], (1, 1, S, S), {"starts": [0], "ends": [S], "axes": [3]}, "bool")
        s = b.op("Where", [b.cast(m, "bool"), b.cast(s, dt), mask_value], b.shape(s))
        s = b.ew("Add", s, em)
        if dt != "f32":
            s = b.cast(s, "f32")
            b.dtype = "f32"
        e = b.ew("Exp", b.ew("Sub", s, b.reduce("ReduceMax", s)))
        p = b.ew("Div", e, b.reduce("ReduceSum", e))
        b.dtype = dt
        if dt != "f32":
            p = b.cast(p, dt)
        o = b.reshape(b.transpose(b.matmul(p, v, causal), (0, 2, 1, 3)), (B, S, D))
        h = b.ew("Add", h, lin(f"l{l}_proj", o, D, D))
        f = _gelu_tanh(b, lin(f"l{l}_fc", _layernorm(b, h, D, f"l{l}_ln2", True), D, F), f"l{l}_gelu")
        h = b.ew("Add", h, lin(f"l{l}_fcproj", f, F, D))
    b.output(b.matmul(_layernorm(b, h, D, "lnf", True), b.transpose(wte, (1, 0))))
    return b


def unet_decoder(c):
    """Per step: pointwise convolution, 2x nearest-neighbour Resize, Concat with a skip map, 3x3 convolution."""
    N, ch, r = c["N"], c["C"], c["R"]
    b = _Net(c["dtype"])
    x = b.input("x", (N, ch, r, r), _normal())
    for i in range(c["steps"]):
        half = ch // 2
        skip = b.input(f"skip{i}", (N, half, 2 * r, 2 * r), _normal())

        def conv(name, t, k):
            w = b.weight(f"{name}_w", (half, ch, k, k), _normal(0.0, math.sqrt(2.0 / (ch * k * k))))
            return b.ew("Relu", b.conv(t, w, b.weight(f"{name}_b", (half,), _normal(0.0, 0.1)), 1, k // 2))

        t = b.op("Resize", [conv(f"up{i}", x, 1)], (N, half, 2 * r, 2 * r), {"scales": [1, 1, 2, 2]})
        x = conv(f"mix{i}", b.op("Concat", [t, skip], (N, ch, 2 * r, 2 * r), {"axis": 1}), 3)
        ch, r = half, 2 * r
    b.output(x)
    return b


GRAPHS = {f.__name__: f for f in (residual_block, resnet_stage, memory_bound_chain, encoder_layer, efficientnet, decoder, unet_decoder)}


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # one residual block on one image: a single kernel, all latency
        dict(name="residual_f32", graph="residual_block", N=1, C=64, H=56, W=56, dtype="f32", tuned=True),
        # the One-to-One chain with channel shuffle over a batch of maps, and over a small, odd-sized one
        dict(name="chain_f32", graph="memory_bound_chain", N=16, C=256, H=64, W=64, groups=8, rounds=3, dtype="f32", tuned=True),
        dict(name="chain_f32_odd", graph="memory_bound_chain", N=3, C=48, H=37, W=29, groups=4, rounds=3, dtype="f32"),
        # dense 3x3 convolutions, batched inference
        dict(name="resnet_f16", graph="resnet_stage", N=32, C=64, R=56, dtype="f16", layout=1),
        # a decoder half of a segmentation network: upsampling, concatenation, 3x3 convolutions
        dict(name="unet_f16", graph="unet_decoder", N=8, C=256, R=16, steps=3, dtype="f16", layout=1),
        # image classification backbone, batched, served with the extended plan; and a single image with the table's plan
        dict(name="efficientnet_f16_b32", graph="efficientnet", N=32, R=224, stages=7, dtype="f16", layout=1, extensions=True, tuned=True),
        dict(name="efficientnet_f16_b1", graph="efficientnet", N=1, R=224, stages=7, dtype="f16", layout=1),
        # encoder layer: batched serving; one short request of ragged length; full precision
        dict(name="encoder_f16_b8", graph="encoder_layer", B=8, S=384, D=768, NH=12, F=3072, dtype="f16", attention=1, tuned=True),
        dict(name="encoder_bf16_b1_s77", graph="encoder_layer", B=1, S=77, D=768, NH=12, F=3072, dtype="bf16"),
        dict(name="encoder_f32_b2_s128", graph="encoder_layer", B=2, S=128, D=768, NH=12, F=3072, dtype="f32"),
        # decoder stack: the headline workload (the largest case), and one short prompt
        dict(name="decoder_bf16_b4_s1024", graph="decoder", B=4, S=1024, D=768, NH=12, L=12, V=50257, dtype="bf16", tuned=True),
        dict(name="decoder_bf16_b1_s33", graph="decoder", B=1, S=33, D=768, NH=12, L=12, V=50257, dtype="bf16", attention=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Drawn shapes are planned without tuning on the device: tuning compiles every tile form of every product, about a
    minute for a shape that has not been seen before."""
    graph = rng.choice(sorted(GRAPHS))
    c = dict(graph=graph, dtype=rng.choice(["f16", "bf16"]))
    if graph == "residual_block":
        c.update(dtype=rng.choice(["f32", "f16", "bf16"]), N=_log(rng, 1, 16), C=rng.choice([16, 24, 32, 40, 64, 96, 128]),
                 H=rng.randint(7, 80), W=rng.randint(7, 80))
    elif graph == "resnet_stage":
        c.update(N=_log(rng, 1, 32), C=rng.choice([16, 32, 48, 64]), R=rng.randint(20, 80), layout=int(rng.random() < 0.75))
    elif graph == "memory_bound_chain":
        c.update(dtype="f32", N=_log(rng, 1, 16), C=8 * rng.randint(2, 32), H=rng.randint(7, 64), W=rng.randint(7, 64), groups=rng.choice([2, 4, 8]), rounds=rng.randint(1, 3))
    elif graph == "unet_decoder":
        c.update(N=_log(rng, 1, 8), C=rng.choice([32, 64, 128, 256]), R=rng.randint(6, 24), steps=rng.randint(2, 3), layout=int(rng.random() < 0.75))
    elif graph == "efficientnet":
        c.update(N=_log(rng, 1, 32), R=rng.randint(64, 224), stages=rng.randint(2, 5), layout=int(rng.random() < 0.75))
        c.update(extensions=bool(c["layout"] and rng.random() < 0.5))
    elif graph == "encoder_layer":
        D, NH = rng.choice([(128, 4), (256, 4), (384, 6), (768, 12)])
        c.update(dtype=rng.choice(["f16", "bf16", "f32"]), B=_log(rng, 1, 16), S=_log(rng, 16, 512), D=D, NH=NH, F=4 * D)
        c.update(attention=int(c["dtype"] != "f32" and rng.random() < 0.5))
    else:
        D, NH = rng.choice([(128, 4), (384, 6), (768, 12)])
        S = _log(rng, 8, 1024)
        c.update(B=max(1, min(_log(rng, 1, 8), 4096 // S)), S=S, D=D, NH=NH, L=rng.randint(1, 12), V=rng.choice([211, 1003, 50257]), attention=rng.randint(0, 1))
    return c


def work(case):
    b = GRAPHS[case["graph"]](case)
    return {"bytes": b.bytes(), "flops": b.flops}


def tolerance(case):
    """Four times what correct plans of one graph differ by on the same values (the operators one by one against fused
    blocks, channels-last against the declared order, streaming softmax against stored scores): relative to the result
    5e-7 at most in f32, 0.7-1.8e-3 in f16, 2-9e-3 in bf16 and 0.010-0.015 after the decoder's twelve layers."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-5}
    if case["dtype"] == "f16":
        return {"rel": 4e-3, "max": 3e-2}
    return {"rel": 3e-2, "max": 0.3} if case["graph"] == "decoder" else {"rel": 2e-2, "max": 0.15}


def prepare(case, seed):
    b = GRAPHS[case["graph"]](case)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    g = api.Graph()
    ids, bufs = {}, {"input": [], "weight": [], "output": []}
    for name, (dtype, shape, kind, fill, value) in b.tensors.items():
        ids[name] = g.add_tensor(name, dtype, shape, kind)
        if value is not None:
            g.set_const(ids[name], value)
        if fill is not None:
            bufs[kind].append(fill(gen, shape).to(dev, TORCH_TYPES[dtype]).contiguous())
        elif kind == "output":
            bufs[kind].append(torch.empty(shape, dtype=TORCH_TYPES[dtype], device=dev))
    for kind, ins, outs, attrs in b.ops:
        g.add_op(kind, [ids[i] for i in ins], [ids[o] for o in outs], attrs)
    g.finalize()
    g.rewrite()
    opts = {k: case[k] for k in ("layout", "attention") if k in case}
    if case.get("extensions"):
        opts.update(broadcast_prologue=1, squeeze_excite=2)
    stream = torch.cuda.current_stream(dev).cuda_stream
    scratch = None
    if case.get("tuned"):
        scratch = torch.zeros(PROFILE_BYTES, dtype=torch.uint8, device=dev)
        opts.update(profile=1, tune=1, profile_scratch=scratch.data_ptr(), profile_scratch_bytes=scratch.numel())
    plan = api.Plan(g, [w.data_ptr() for w in bufs["weight"]], stream=stream, cache_dir=CACHE, **opts)
    workspace = torch.empty(max(plan.workspace_bytes(), 256), dtype=torch.uint8, device=dev)
    plan.prepare(workspace.data_ptr(), stream)
    return {"plan": plan, "workspace": workspace, "weights": bufs["weight"], "inputs": bufs["input"], "outputs": bufs["output"]}


def run(state):
    state["plan"].run([t.data_ptr() for t in state["inputs"]], [t.data_ptr() for t in state["outputs"]],
                      state["workspace"].data_ptr(), torch.cuda.current_stream().cuda_stream)
    return state["outputs"]
