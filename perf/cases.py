"""The work a program has this library do, as cases that can be timed and compared.

A cold inference of a convolutional network is, per layer, the transformation of the raw weights
and the execution of the kernel chosen for it; a program calls this library for one layer
(`nnv_conv_forward*`), for the weights of a whole model (`nnv_transform_weights_grouped`), for many
layers at once (`nnv_conv_forward_grouped`) and for a whole cold pass (`nnv_cold_stack`).  The cases
cover those four, float32 and float16 storage, every kernel kind, and sizes from a single 16-channel
layer to whole stacks and batches; the layer shapes are those of `nnv_workloads` at any input
resolution and batch, and free single layers.

Inputs: weights He-normal, activations U(-1, 1), biases N(0, 0.1^2), as everywhere in this
repository, drawn on the GPU from the seed alone.
"""
import math
from dataclasses import replace

import torch

import paper_2206_07446_amd as nnv
from nnv_workloads import ConvLayer, STACK_NAMES, stack

KIND = nnv.KINDS


def listed():
    return [
        # The smallest call: one thin layer on a small map, where the call itself is the cost.
        dict(name="layer_small", op="layer", kind="im2col_gemm", dtype="f32", n=1, c=16, h=32, w=32, k=16, r=3, stride=1,
             pad=1, groups=1, relu=False),
        # An ordinary layer of an inception network as a serving program runs it: few images, channel
        # counts that fill no tile, half-precision storage, bias and activation in the same call.
        dict(name="layer_f16_ragged", op="layer", kind="wino_f4", dtype="f16", n=3, c=96, h=14, w=14, k=208, r=3, stride=1,
             pad=1, groups=1, relu=True),
        # A large layer at a throughput batch.
        dict(name="layer_f32_batch8", op="layer", kind="im2col_gemm", dtype="f32", n=8, c=256, h=56, w=56, k=256, r=3,
             stride=1, pad=1, groups=1, relu=True),
        # The weights of a model at cold start for every kernel candidate: what the decision stage needs.
        dict(name="transform_resnet18_all", op="transform", stack="resnet18", kind="all", dtype="f32"),
        # The weights of a larger model in half precision, into the layouts of the kinds it would execute with.
        dict(name="transform_resnet50_f16", op="transform", stack="resnet50", kind="gemm+f4", dtype="f16"),
        # All layers of a network by one kernel candidate (the decision stage's execution profile), batch 1.
        dict(name="direct_resnet18", op="grouped", stack="resnet18", kind="direct", dtype="f32", n=1, h=224, w=224, relu=False),
        dict(name="gemm_resnet18", op="grouped", stack="resnet18", kind="im2col_gemm", dtype="f32", n=1, h=224, w=224, relu=False),
        dict(name="f2_resnet18", op="grouped", stack="resnet18", kind="wino_f2", dtype="f32", n=1, h=224, w=224, relu=False),
        # A mobile network by its plan: depthwise layers in the depthwise kind, the others by implicit GEMM.
        dict(name="plan_mobilenetv2", op="grouped", stack="mobilenetv2", kind="plan", dtype="f32", n=1, h=224, w=224, relu=True),
        # A network of wide 3x3 layers by Winograd, the largest transformed weights.
        dict(name="f4_vgg16", op="grouped", stack="vgg16", kind="wino_f4", dtype="f32", n=1, h=224, w=224, relu=True),
        # A deep network of bottlenecks in half precision.
        dict(name="gemm_resnet50_f16", op="grouped", stack="resnet50", kind="im2col_gemm", dtype="f16", n=1, h=224, w=224, relu=True),
        # The cold pass itself: raw weights to outputs, layer after layer, a layer reading what the one
        # before it wrote wherever the shapes let it.
        dict(name="cold_resnet18", op="cold", stack="resnet18", kind="plan", dtype="f32", n=1, h=224, w=224, stage_layers=0,
             streams=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    op = rng.choice(("layer", "layer", "grouped", "grouped", "grouped", "transform", "cold"))
    dtype = rng.choice(("f32", "f32", "f16"))
    if op == "layer":
        kind = rng.choice(("direct", "im2col_gemm", "im2col_gemm", "wino_f2", "wino_f4", "wino_f6", "depthwise"))
        r, stride = 3, 1
        if kind in ("direct", "im2col_gemm"):
            r, stride = rng.choice(((1, 1), (1, 2), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2)))
        elif kind == "depthwise":
            r, stride = rng.choice((3, 3, 5)), rng.choice((1, 2))
        c, k = _log(rng, 3, 1024), _log(rng, 8, 1024)
        groups = 1
        if kind == "depthwise":
            k = groups = c
        elif kind in ("direct", "im2col_gemm") and rng.random() < 0.1:
            groups = rng.choice((2, 3, 4))
            c, k = groups * _log(rng, 8, 256), groups * _log(rng, 8, 256)
        return dict(op=op, kind=kind, dtype=dtype, n=_log(rng, 1, 16), c=c, h=_log(rng, 7, 224), w=_log(rng, 7, 224), k=k, r=r,
                    stride=stride, pad=r // 2, groups=groups, relu=rng.random() < 0.5)
    name = rng.choice(STACK_NAMES)
    if op == "transform":
        return dict(op=op, stack=name, kind=rng.choice(("all", "plan", "gemm+f4", "wino_f2", "wino_f4")), dtype=dtype)
    d = dict(op=op, stack=name, kind="plan", dtype=dtype, n=_log(rng, 1, 4), h=rng.randint(96, 320), w=rng.randint(96, 320))
    if op == "cold":
        d.update(kind=rng.choice(("plan", "plan", "direct")), stage_layers=rng.choice((0, 0, 1, 4)), streams=rng.choice((1, 1, 2)))
    else:
        d.update(kind=rng.choice(("direct", "im2col_gemm", "wino_f2", "wino_f4", "wino_f6", "plan")), relu=rng.random() < 0.5)
    return d


_MOST_FLOPS = {"direct": 4e9}   # the vector kernels take as long for these as the others for 16e9
_MOST_BYTES = 4e8


def draw(rng):
    while True:
        case = _draw(rng)
        layers, kinds = _layers(case)
        if not layers:
            continue
        w = work(case)
        if w["flops"] <= _MOST_FLOPS.get(case["kind"], 16e9) and w["bytes"] <= _MOST_BYTES:
            return case


# ---- shapes

def _dtype(case):
    return nnv.F16 if case["dtype"] == "f16" else nnv.F32


def _ok(layer, kind, dtype):
    return nnv.nnv_kind_supported(nnv.make_desc(layer, dtype), kind)


def _scaled(layers, case):
    """The stack at another input size and batch (maps of 1x1 behind a global pool stay as they are)."""
    def size(v, to, r, pad):
        return v if v == 1 else max(r - 2 * pad, 1, -(-v * to // 224))
    return [replace(l, h=size(l.h, case["h"], l.r, l.pad), w=size(l.w, case["w"], l.s, l.pad), n=case["n"]) for l in layers]


def _plan_kind(layer, dtype):
    for kind in (nnv.DEPTHWISE, nnv.IM2COL_GEMM):
        if _ok(layer, kind, dtype):
            return kind
    return nnv.DIRECT


def _layers(case):
    """The (layer, kind) pairs of a case: two lists."""
    dtype, kind = _dtype(case), case["kind"]
    if case["op"] == "layer":
        layer = ConvLayer("layer", case["c"], case["h"], case["w"], case["k"], case["r"], case["r"], case["stride"], case["pad"],
                          case["groups"], case["n"])
        return ([layer], [KIND[kind]]) if _ok(layer, KIND[kind], dtype) else ([], [])
    layers = stack(case["stack"])
    if case["op"] != "transform":
        layers = _scaled(layers, case)
    if kind == "plan":
        pairs = [(l, _plan_kind(l, dtype)) for l in layers]
        if case["op"] == "transform":
            pairs = [(l, k) for l, k in pairs if k != nnv.DIRECT]
    else:
        wanted = {"all": ("im2col_gemm", "wino_f2", "wino_f4", "depthwise"), "gemm+f4": ("im2col_gemm", "wino_f4")}.get(kind, (kind,))
        pairs = [(l, KIND[k]) for l in layers for k in wanted if _ok(l, KIND[k], dtype)]
    return [l for l, _ in pairs], [k for _, k in pairs]


def _esz(case):
    return 2 if case["dtype"] == "f16" else 4


def _x_elems(l):
    return l.n * l.c * l.h * l.w


def _y_elems(l):
    return l.n * l.k * l.p * l.q


def _flops(l, kind):
    m = {nnv.WINO_F2: 2, nnv.WINO_F4: 4, nnv.WINO_F6: 6}.get(kind)
    if m:
        return 2.0 * (m + 2) ** 2 * l.k * l.c * l.n * -(-l.p // m) * -(-l.q // m)
    return 2.0 * l.macs


# ---- state

class _Flat:
    """Many tensors in one allocation, each on a 256-byte boundary."""

    def __init__(self, byte_sizes, device):
        self.at, total = [], 0
        for b in byte_sizes:
            self.at.append((total, b))
            total += -(-b // 256) * 256
        self.all = torch.zeros(max(total, 256), dtype=torch.uint8, device=device)

    def views(self, dtype):
        return [self.all[o:o + b].view(dtype) for o, b in self.at]


def prepare(case, seed):
    dev = torch.device("cuda")
    dtype = _dtype(case)
    store = torch.float16 if dtype == nnv.F16 else torch.float32
    layers, kinds = _layers(case)
    descs = [nnv.make_desc(l, dtype) for l in layers]
    gen = torch.Generator(device=dev).manual_seed(seed)
    raws, by_layer = [], {}
    for l in layers:
        if l.name not in by_layer:   # the candidates of one layer transform the same raw weights
            by_layer[l.name] = torch.randn(l.params, device=dev, generator=gen).mul_(math.sqrt(2.0 / (l.cg * l.r * l.s)))
        raws.append(by_layer[l.name])
    # the direct kind executes from the raw weights: nothing to transform
    sizes = [0 if k == nnv.DIRECT else nnv.nnv_transformed_bytes(d, k) for d, k in zip(descs, kinds)]
    tx = _Flat(sizes, dev)
    wt = [raw if k == nnv.DIRECT else t for raw, k, t in zip(raws, kinds, tx.views(torch.uint8))]
    s = {"op": case["op"], "descs": descs, "kinds": kinds, "raws": raws, "wt": wt, "tx": tx.all.view(store)}
    if case["op"] == "transform":
        return s
    ys = _Flat([_y_elems(l) * _esz(case) for l in layers], dev)
    s["ys"], s["y"] = ys.views(store), ys.all.view(store)
    xs = []
    for i, l in enumerate(layers):
        before = layers[i - 1] if i else None
        if case["op"] == "cold" and before and (before.n, before.k, before.p, before.q) == (l.n, l.c, l.h, l.w):
            xs.append(s["ys"][i - 1])
        else:
            xs.append(torch.rand(_x_elems(l), device=dev, generator=gen).mul_(2).sub_(1).to(store))
    s["xs"] = xs
    if case["op"] == "cold":
        need = max(nnv.nnv_workspace_bytes(d, k) for d, k in zip(descs, kinds))
        s["stage_layers"] = case["stage_layers"]
        s["stream_tx"] = torch.cuda.Stream() if case["streams"] == 2 else None
    else:
        s["relu"] = case["relu"]
        s["bias"] = [torch.randn(l.k, device=dev, generator=gen).mul_(0.1) if case["relu"] else None for l in layers]
        nnv.nnv_transform_weights_grouped(*_to_transform(s))
        need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
        if case["op"] == "layer":
            need = nnv.nnv_workspace_bytes(descs[0], kinds[0])
    s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
    return s


def _to_transform(s):
    todo = [i for i, k in enumerate(s["kinds"]) if k != nnv.DIRECT]
    return [[s[key][i] for i in todo] for key in ("descs", "kinds", "raws", "wt")]


def run(s):
    op = s["op"]
    if op == "layer":
        call = nnv.nnv_conv_forward_relu if s["relu"] else nnv.nnv_conv_forward
        call(s["descs"][0], s["kinds"][0], s["xs"][0], s["wt"][0], s["bias"][0], s["ys"][0], s["ws"])
        return s["y"]
    if op == "transform":
        nnv.nnv_transform_weights_grouped(s["descs"], s["kinds"], s["raws"], s["wt"])
        return s["tx"]
    if op == "grouped":
        nnv.nnv_conv_forward_grouped(s["descs"], s["kinds"], s["xs"], s["wt"], s["bias"] if s["relu"] else None, s["ys"], s["ws"],
                                     flags=nnv.FORWARD_RELU if s["relu"] else 0)
        return s["y"]
    nnv.nnv_cold_stack(s["descs"], s["kinds"], s["raws"], s["wt"], s["xs"], s["ys"], s["ws"], stage_layers=s["stage_layers"],
                       stream_tx=s["stream_tx"])
    return {"y": s["y"], "w": s["tx"]}


def work(case):
    layers, kinds = _layers(case)
    raw = {l.name: 4 * l.params for l in layers}
    tx = [nnv.nnv_transformed_bytes(nnv.make_desc(l, _dtype(case)), k) for l, k in zip(layers, kinds)]
    acts = _esz(case) * sum(_x_elems(l) + _y_elems(l) for l in layers)
    if case["op"] == "transform":
        return {"bytes": sum(raw.values()) + sum(tx), "flops": 0}
    if case["op"] == "cold":   # the transformed weights are written, then executed from
        written = sum(t for t, k in zip(tx, kinds) if k != nnv.DIRECT)
        return {"bytes": sum(raw.values()) + written + acts, "flops": sum(map(_flops, layers, kinds))}
    return {"bytes": sum(tx) + acts, "flops": sum(map(_flops, layers, kinds))}


def tolerance(case):
    kinds = set(_layers(case)[1])
    if case["op"] == "transform":
        if kinds <= {nnv.IM2COL_GEMM, nnv.DEPTHWISE}:
            return "exact"   # index permutations, one rounding to the storage type
        # a handful of float32 roundings per value; float16 storage adds one that may fall either way
        return {"rel": 2e-4} if case["dtype"] == "f16" else {"rel": 1e-6}
    if case["dtype"] == "f16":
        # one rounding of y that may fall either way; Winograd rounds its transformed input as well
        rel = {nnv.WINO_F2: 1e-3, nnv.WINO_F4: 3e-3}
        return {"rel": max(rel.get(k, 5e-4) for k in kinds)}
    # float32 sums of up to some thousand terms in any order; the tile transforms of F(4x4) and F(6x6) amplify roundings
    rel = {nnv.WINO_F4: 2e-5, nnv.WINO_F6: 5e-5}
    return {"rel": max(rel.get(k, 1e-5) for k in kinds)}
