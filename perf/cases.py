"""Performance cases: the calls a program makes to this engine, over the range of sizes it is used at.

A case is one network or part of a network, given to ``engine.Plan`` as an operator list and run with
``Plan.run`` (or ``Plan.capture`` once and ``Plan.replay`` per call).  Most cases are single layers and
blocks, each a plan of its own that takes NHWC features and returns NHWC fp32 values, as a program does
that runs a backbone stage or a head by itself; two are whole networks.  Sizes are those of MobileNet v1
and v2 and of the dense-prediction head at their usual resolutions, and odd ones between them.

Keys of a case:
  kind     separable | inverted | front | conv | head | dense_head | v1 | v2 (see ``network``)
  n, h, w  batch and input plane;  c: input channels;  cout: output channels (classes for a head)
  k, s     window and stride of the (first) depthwise or full convolution
  depth    separable: number of chained layers;  e: inverted: expansion factor
  store    storage type of activations and weights, fp16 or bf16;  src: element type of the input, fp16 or fp32
  tune     Plan.autotune before use;  graph: a captured plan, replayed
"""
import math

import numpy as np
import torch

from paper_1907_01989_amd import _binding as B
from paper_1907_01989_amd import engine

NONE, RELU, RELU6 = 0, 1, 2

BASE = {"k": 3, "s": 1, "depth": 1, "e": 6, "store": "fp16", "src": "fp16", "tune": False, "graph": False}


def _case(**kw):
    return {**BASE, **kw}


def listed():
    return [
        # one depthwise-separable layer on one image: the benchmark's block workload; the smallest call, where
        # launches and latency count
        _case(name="separable56_b1", kind="separable", n=1, h=56, w=56, c=128, cout=128),
        # v1's five equal 14x14x512 layers run as a backbone stage at the serving batch
        _case(name="separable14x5_b64", kind="separable", n=64, h=14, w=14, c=512, cout=512, depth=5),
        # a down-sampling layer at a small batch, bf16 storage, fp32 features from another framework
        _case(name="separable28s2_b8_bf16", kind="separable", n=8, h=28, w=28, c=256, cout=512, s=2, store="bf16", src="fp32"),
        # a depthwise layer with a larger window (any window is supported), mid batch
        _case(name="separable28k5_b16", kind="separable", n=16, h=28, w=28, c=240, cout=80, k=5),
        # v2's residual block at 28x28
        _case(name="inverted28_b32", kind="inverted", n=32, h=28, w=28, c=32, cout=32),
        # v2's strided 96 -> 160 block on an odd plane and an odd batch, bf16 storage
        _case(name="inverted15s2_b5_bf16", kind="inverted", n=5, h=15, w=15, c=96, cout=160, s=2, store="bf16", src="fp32"),
        # the first three layers on fp32 images at the 192 resolution
        _case(name="front192_b16", kind="front", n=16, h=192, w=192, c=3, cout=64, src="fp32"),
        # a full 3x3 convolution on the dense-prediction feature size
        _case(name="conv33_b4", kind="conv", n=4, h=33, w=33, c=256, cout=256),
        # v1's classifier: last pointwise layer, pool, fully connected, softmax
        _case(name="head7_b64", kind="head", n=64, h=7, w=7, c=1024, cout=1000),
        # the dense-prediction head: two branches, concat, logits, x16 upsampling and labels, odd plane
        _case(name="dense_head33_b2", kind="dense_head", n=2, h=33, w=33, c=320, cout=21),
        # the whole v1 network at the benchmark's batch, tuned as the benchmark does: the largest call
        _case(name="v1_224_b64", kind="v1", n=64, h=224, w=224, c=3, cout=1000, tune=True),
        # the whole v2 network on one image as an interactive program runs it: one captured graph per call
        _case(name="v2_224_b1", kind="v2", n=1, h=224, w=224, c=3, cout=1000, graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["separable", "separable", "separable", "inverted", "inverted", "front", "conv", "head",
                           "dense_head", "v1", "v2"])
        c = _case(kind=kind, n=_log(rng, 1, 64), store=rng.choice(["fp16", "fp16", "bf16"]), src=rng.choice(["fp16", "fp32"]))
        if kind == "separable":
            c["h"] = _log(rng, 5, 112)
            c["w"] = c["h"] + rng.choice([0, 0, 0, -1, 2])
            c["c"] = max(8, 8 * _log(rng, 2, 128) - rng.choice([0, 0, 0, 3]))
            c["k"] = rng.choice([3, 3, 3, 3, 5])
            c["s"] = rng.choice([1, 1, 2])
            c["depth"] = rng.choice([1, 1, 2, 3, 5]) if c["s"] == 1 else 1
            c["cout"] = c["c"] if c["depth"] > 1 or c["s"] == 1 and rng.random() < 0.5 else 8 * _log(rng, 2, 128)
        elif kind == "inverted":
            c["h"] = _log(rng, 5, 112)
            c["w"] = c["h"] + rng.choice([0, 0, 0, -1, 2])
            c["c"] = 8 * _log(rng, 2, 40)
            c["s"] = rng.choice([1, 1, 2])
            c["cout"] = c["c"] if c["s"] == 1 and rng.random() < 0.7 else 8 * _log(rng, 2, 40)
            c["e"] = rng.choice([3, 4, 6, 6])
        elif kind == "front":
            c["h"] = _log(rng, 96, 321)
            c["w"], c["c"], c["cout"] = c["h"], 3, rng.choice([16, 32, 64])
        elif kind == "conv":
            c["h"] = _log(rng, 7, 65)
            c["w"] = c["h"] + rng.choice([0, 0, -1, 2])
            c["c"], c["cout"] = 8 * _log(rng, 4, 64), 8 * _log(rng, 2, 64)
            c["s"] = rng.choice([1, 1, 2])
        elif kind == "head":
            c["h"] = rng.choice([3, 4, 5, 6, 7, 7, 8])
            c["w"], c["c"], c["cout"] = c["h"], rng.choice([256, 320, 512, 1024]), _log(rng, 10, 1000)
        elif kind == "dense_head":
            c["n"] = _log(rng, 1, 8)
            c["h"] = rng.choice([17, 21, 25, 29, 33, 33, 41])
            c["w"], c["c"], c["cout"] = c["h"], rng.choice([256, 320]), rng.choice([2, 19, 21, 21])
        else:
            c["n"] = _log(rng, 1, 64 if kind == "v1" else 24)
            c["h"] = rng.choice([96, 128, 160, 192, 192, 224, 224, 225])
            c["w"], c["c"], c["cout"] = c["h"], 3, 1000
            c["store"] = "fp16"
            mode = rng.choice(["", "", "tune", "graph"])
            c["tune"], c["graph"] = mode == "tune", mode == "graph"
        ops, _ = network(c)
        moved = sum(2 * _elems(op) for op in ops)
        macs = sum(_macs(op, ops) for op in ops)
        whole = kind in ("v1", "v2")
        if whole and c["n"] * c["h"] * c["h"] <= (64 if kind == "v1" else 24) * 224 * 224 or \
                not whole and moved <= 150e6 and macs <= 20e9:
            return c


# ------------------------------------------------------------------- networks
def _same(size, k, s, d=1):
    out = -(-size // s)
    total = max((out - 1) * s + (k - 1) * d + 1 - size, 0)
    return total // 2, total - total // 2, out


class _Net:
    """Operator list of a network; ``rng`` draws its weights (none: shapes only)."""

    def __init__(self, rng, store):
        self.ops, self.outputs, self.rng, self.store = [], [], rng, store

    def _push(self, op, shape):
        op["out"] = tuple(shape)
        self.ops.append(op)
        return len(self.ops) - 1

    def _weights(self, shape, fan_in, cout):
        if self.rng is None:
            return None, None
        w = torch.from_numpy(self.rng.standard_normal(shape, dtype=np.float32) * np.float32(math.sqrt(2.0 / fan_in)))
        w = w.to(torch.float16 if self.store == "fp16" else torch.bfloat16).float().numpy()
        return w, self.rng.standard_normal(cout, dtype=np.float32) * np.float32(0.01)

    def input(self, n, h, w, c, dtype):
        return self._push({"op": "input", "shape": (n, h, w, c), "dtype": dtype}, (n, h, w, c))

    def conv(self, x, cout, k=1, s=1, act=RELU6):
        n, h, w, cin = self.ops[x]["out"]
        pt, pb, oh = _same(h, k, s)
        pl, pr, ow = _same(w, k, s)
        wt, b = self._weights((cout, k, k, cin), k * k * cin, cout)
        return self._push({"op": "conv2d", "in": x, "kh": k, "kw": k, "stride": (s, s), "dil": (1, 1),
                           "pads": (pt, pb, pl, pr), "cout": cout, "act": act, "w": wt, "b": b}, (n, oh, ow, cout))

    def dw(self, x, k=3, s=1, act=RELU6):
        n, h, w, c = self.ops[x]["out"]
        pt, pb, oh = _same(h, k, s)
        pl, pr, ow = _same(w, k, s)
        wt, b = self._weights((c, k, k), k * k, c)
        return self._push({"op": "depthwise", "in": x, "kh": k, "kw": k, "stride": (s, s), "dil": (1, 1),
                           "pads": (pt, pb, pl, pr), "act": act, "w": wt, "b": b}, (n, oh, ow, c))

    def add(self, a, b):
        return self._push({"op": "add", "a": a, "b": b, "act": NONE}, self.ops[a]["out"])

    def gap(self, x):
        n, _, _, c = self.ops[x]["out"]
        return self._push({"op": "gap", "in": x}, (n, 1, 1, c))

    def fc(self, x, cout):
        n, _, _, c = self.ops[x]["out"]
        wt, b = self._weights((cout, c), c, cout)
        return self._push({"op": "fc", "in": x, "cout": cout, "w": wt, "b": b}, (n, 1, 1, cout))

    def softmax(self, x):
        return self._push({"op": "softmax", "in": x}, self.ops[x]["out"])

    def concat(self, xs):
        n, h, w, _ = self.ops[xs[0]]["out"]
        return self._push({"op": "concat", "ins": list(xs)}, (n, h, w, sum(self.ops[t]["out"][3] for t in xs)))

    def resize(self, x, oh, ow):
        n, _, _, c = self.ops[x]["out"]
        return self._push({"op": "resize_bilinear", "in": x, "oh": oh, "ow": ow, "align_corners": 1}, (n, oh, ow, c))

    def argmax(self, x):
        n, h, w, _ = self.ops[x]["out"]
        return self._push({"op": "argmax", "in": x}, (n, h, w, 1))


def network(case, rng=None):
    """(ops, outputs) of a case; weights come from ``rng``."""
    g = _Net(rng, case["store"])
    kind, cout = case["kind"], case["cout"]
    t = g.input(case["n"], case["h"], case["w"], case["c"], B.DTYPE_FP16 if case["src"] == "fp16" else B.DTYPE_FP32)
    if kind == "separable":
        for i in range(case["depth"]):
            t = g.dw(t, case["k"], case["s"] if i == 0 else 1)
            t = g.conv(t, cout)
        outs = [t]
    elif kind == "inverted":
        y = g.conv(t, case["c"] * case["e"])
        y = g.dw(y, 3, case["s"])
        y = g.conv(y, cout, act=NONE)
        outs = [g.add(y, t) if case["s"] == 1 and cout == case["c"] else y]
    elif kind == "front":
        t = g.conv(t, 32, 3, 2)
        t = g.dw(t)
        outs = [g.conv(t, cout)]
    elif kind == "conv":
        outs = [g.conv(t, cout, case["k"], case["s"])]
    elif kind == "head":
        t = g.conv(t, 1024)
        z = g.fc(g.gap(t), cout)
        outs = [z, g.softmax(z)]
    elif kind == "dense_head":
        a = g.conv(t, 256, act=RELU)
        p = g.conv(g.gap(t), 256, act=RELU)
        z = g.conv(g.concat([a, g.resize(p, case["h"], case["w"])]), cout, act=NONE)
        outs = [z, g.argmax(g.resize(z, 16 * (case["h"] - 1) + 1, 16 * (case["w"] - 1) + 1))]
    elif kind == "v1":
        t = g.conv(t, 32, 3, 2)
        for c, s in [(64, 1), (128, 2), (128, 1), (256, 2), (256, 1), (512, 2), (512, 1), (512, 1), (512, 1), (512, 1),
                     (512, 1), (1024, 2), (1024, 1)]:
            t = g.conv(g.dw(t, 3, s), c)
        z = g.fc(g.gap(t), cout)
        outs = [z, g.softmax(z)]
    else:
        t = g.conv(t, 32, 3, 2)
        cin = 32
        for e, c, reps, s0 in [(1, 16, 1, 1), (6, 24, 2, 2), (6, 32, 3, 2), (6, 64, 4, 2), (6, 96, 3, 1), (6, 160, 3, 2),
                               (6, 320, 1, 1)]:
            for r in range(reps):
                s = s0 if r == 0 else 1
                y = g.conv(t, cin * e) if e != 1 else t
                y = g.conv(g.dw(y, 3, s), c, act=NONE)
                t = g.add(y, t) if s == 1 and cin == c else y
                cin = c
        z = g.fc(g.gap(g.conv(t, 1280)), cout)
        outs = [z, g.softmax(z)]
    return g.ops, outs


def _elems(op):
    return math.prod(op["out"])


def _macs(op, ops):
    if op["op"] == "conv2d":
        return _elems(op) * op["kh"] * op["kw"] * ops[op["in"]]["out"][3]
    if op["op"] == "depthwise":
        return _elems(op) * op["kh"] * op["kw"]
    if op["op"] == "fc":
        return _elems(op) * ops[op["in"]]["out"][3]
    return 0


def _nweights(op, ops):
    if op["op"] == "conv2d":
        return op["cout"] * op["kh"] * op["kw"] * ops[op["in"]]["out"][3]
    if op["op"] == "depthwise":
        return op["kh"] * op["kw"] * op["out"][3]
    if op["op"] == "fc":
        return op["cout"] * ops[op["in"]]["out"][3]
    return 0


def work(case):
    """The input read once, the outputs written once (fp32 or int32), the weights read once in their storage type."""
    ops, outs = network(case)
    nbytes = _elems(ops[0]) * (2 if case["src"] == "fp16" else 4) + sum(4 * _elems(ops[t]) for t in outs)
    nbytes += sum(2 * _nweights(op, ops) for op in ops)
    return {"bytes": nbytes, "flops": 2 * sum(_macs(op, ops) for op in ops)}


# ------------------------------------------------------------ inputs and runs
def _input(case, seed):
    """Images: 8-bit pixels over 255.  Features: what a ReLU6 layer (or, for an inverted block, a linear
    one) hands on."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    shape = (case["n"], case["h"], case["w"], case["c"])
    if case["kind"] in ("front", "v1", "v2"):
        x = torch.randint(0, 256, shape, generator=gen, device="cuda").float() / 255.0
    else:
        x = torch.randn(shape, generator=gen, device="cuda")
        if case["kind"] != "inverted":
            x = (1.5 * x).clamp_(0.0, 6.0)
    return x.to(torch.float16 if case["src"] == "fp16" else torch.float32)


def prepare(case, seed):
    ops, outs = network(case, np.random.default_rng([int(seed), 1]))
    plan = engine.Plan({"ops": ops, "outputs": outs}, dtype=B.DTYPE_FP16 if case["store"] == "fp16" else B.DTYPE_BF16)
    state = {"plan": plan, "x": [_input(case, seed)], "y": plan.alloc_outputs(), "graph": case["graph"]}
    if case["tune"]:
        plan.autotune(state["x"], state["y"])
    if case["graph"]:
        plan.capture(state["x"], state["y"])
    return state


def run(state):
    if state["graph"]:
        return state["plan"].replay()
    return state["plan"].run(state["x"], state["y"])


def tolerance(case):
    """About four times the distance between this engine and the 64-bit result, which is the rounding of each
    stored tensor carried through the layers: 2e-4 to 3e-4 for one layer in fp16, 6e-4 for five, 8 times as
    much in bf16, 4e-4 for v1's logits and 2.4e-3 for v2's.  Labels may differ where two upsampled logits
    nearly tie."""
    if case["kind"] in ("v1", "v2"):
        return {"rel": 2e-3 if case["kind"] == "v1" else 1e-2}
    rel = 1e-3 * (1.0 + 0.2 * (case["depth"] - 1))
    return {"rel": rel if case["store"] == "fp16" else 8 * rel, "differ": 0.005 if case["kind"] == "dense_head" else 0.0}


# -------------------------------------------------------- the result in 64 bits
def _act(x, act):
    return x if act == NONE else x.clamp(min=0) if act == RELU else x.clamp(0, 6)


def _conv64(x, op, depthwise):
    """Convolution of an NHWC tensor as a sum over the window's taps."""
    pt, pb, pl, pr = op["pads"]
    s, (n, oh, ow, cout) = op["stride"][0], op["out"]
    x = torch.nn.functional.pad(x, (0, 0, pl, pr, pt, pb))
    w = torch.from_numpy(op["w"]).to(x)
    y = torch.from_numpy(op["b"]).to(x).expand(n, oh, ow, cout).clone()
    for ky in range(op["kh"]):
        for kx in range(op["kw"]):
            v = x[:, ky:ky + (oh - 1) * s + 1:s, kx:kx + (ow - 1) * s + 1:s]
            y += v * w[:, ky, kx] if depthwise else (v.reshape(-1, v.shape[3]) @ w[:, ky, kx].t().contiguous()).view_as(y)
    return _act(y, op["act"])


def _resize64(x, op):
    _, h, w, _ = x.shape
    _, oh, ow, _ = op["out"]

    def lerp(x, dim, size, out):
        src = torch.arange(out, dtype=torch.float64, device=x.device) * ((size - 1) / (out - 1) if out > 1 else 0.0)
        lo = src.floor().long().clamp(max=size - 1)
        f = (src - lo).view([-1 if d == dim else 1 for d in range(4)])
        return x.index_select(dim, lo) * (1 - f) + x.index_select(dim, (lo + 1).clamp(max=size - 1)) * f

    return lerp(lerp(x, 1, h, oh), 2, w, ow)


def exact(case, seed):
    ops, outs = network(case, np.random.default_rng([int(seed), 1]))
    last, vals, res = {}, {}, {}
    for i, op in enumerate(ops):
        for t in [op[k] for k in ("in", "a", "b") if isinstance(op.get(k), int)] + op.get("ins", []):
            last[t] = i
    for i, op in enumerate(ops):
        k = op["op"]
        if k == "input":
            y = _input(case, seed).double()
        elif k in ("conv2d", "depthwise"):
            y = _conv64(vals[op["in"]], op, k == "depthwise")
        elif k == "add":
            y = _act(vals[op["a"]] + vals[op["b"]], op["act"])
        elif k == "gap":
            y = vals[op["in"]].mean((1, 2), keepdim=True)
        elif k == "fc":
            x = vals[op["in"]]
            y = (x.reshape(x.shape[0], -1) @ torch.from_numpy(op["w"]).to(x).t().contiguous() +
                 torch.from_numpy(op["b"]).to(x)).view(op["out"])
        elif k == "softmax":
            y = vals[op["in"]].softmax(-1)
        elif k == "concat":
            y = torch.cat([vals[t] for t in op["ins"]], 3)
        elif k == "resize_bilinear":
            y = _resize64(vals[op["in"]], op)
        else:
            y = None                                   # labels are whole numbers
        vals[i] = y
        if i in outs:
            n, h, w, c = op["out"]
            res[i] = y if y is None or (h, w) != (1, 1) else y.reshape(n, c)
        for t in [t for t in vals if last.get(t, i) <= i and t != i]:
            del vals[t]
    return [res[t] for t in outs]
