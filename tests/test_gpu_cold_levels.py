"""The convolutions of a cold pass that do not depend on one another share launches: whatever the buffers have in common, the
pass gives, bit for bit, what one layer after the other gives."""
import numpy as np
import pytest

from nnv_workloads import ConvLayer, layer_tensors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2206_07446_amd as nnv
    assert torch.cuda.is_available(), "GPU tests need the HIP device"
    nnv.load()
    return nnv, torch


def Ly(c, h, k, r=3, stride=1, pad=None, groups=1, n=1, w=None):
    return ConvLayer("l", c, h, w or h, k, r, r, stride, r // 2 if pad is None else pad, groups, n)


# every chunking mode, one and two panels per tile, reductions split 1 to 16 ways, more layers than one launch holds, kinds that
# run by themselves in between
LAYERS = [Ly(64, 56, 64), Ly(128, 28, 128), Ly(256, 14, 256), Ly(512, 7, 512), Ly(3, 60, 64, 7, 2), Ly(64, 56, 128, 3, 2),
          Ly(64, 28, 128, 1, 2), Ly(2048, 7, 64, 1), Ly(30, 13, 20, 1), Ly(37, 13, 20, w=19), Ly(16, 27, 48, 5), Ly(20, 12, 16, 4, 1, 2),
          Ly(1, 3, 1), Ly(96, 9, 70, groups=2), Ly(240, 14, 240, 1, groups=3), Ly(16, 32, 16), Ly(8, 9, 24, n=2, w=10), Ly(3, 35, 24, 11, 4, 2),
          Ly(128, 7, 64, n=5), Ly(24, 56, 144, 1), Ly(832, 7, 384, 1), Ly(160, 7, 320), Ly(48, 14, 128, 5), Ly(512, 14, 24, 1),
          Ly(112, 14, 224), Ly(64, 112, 64), Ly(256, 14, 512, 3, 2), Ly(64, 224, 64)]


def tensors(nnv, torch, layers, kinds):
    dev = torch.device("cuda:0")
    descs = [nnv.make_desc(l) for l in layers]
    raw, xs = [], []
    for i, l in enumerate(layers):
        w, x = layer_tensors(l, 900 + i)
        raw.append(torch.from_numpy(w).to(dev)); xs.append(torch.from_numpy(x).to(dev).reshape(-1))
    ws = torch.empty(max([16] + [nnv.nnv_workspace_bytes(d, k) for d, k in zip(descs, kinds)]), dtype=torch.uint8, device=dev)
    wt = [torch.zeros(max(16, nnv.nnv_transformed_bytes(d, k)), dtype=torch.uint8, device=dev) for d, k in zip(descs, kinds)]
    return descs, raw, xs, wt, ws


def one_by_one(nnv, torch, descs, kinds, raw, wt, xs, ys, ws):
    nnv.nnv_transform_weights_grouped(descs, kinds, raw, wt)
    for d, k, t, x, y in zip(descs, kinds, wt, xs, ys):
        nnv.nnv_conv_forward(d, k, x, t, None, y, ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("stage", [0, 5])
def test_independent_layers(env, stage):
    nnv, torch = env
    kinds = [nnv.WINO_F2 if i % 9 == 8 and l.winograd_ok else nnv.IM2COL_GEMM for i, l in enumerate(LAYERS)]
    descs, raw, xs, wt, ws = tensors(nnv, torch, LAYERS, kinds)
    ys = [[torch.full((l.n * l.k * l.p * l.q + 128,), 7.0, device="cuda") for l in LAYERS] for _ in range(2)]
    one_by_one(nnv, torch, descs, kinds, raw, wt, xs, ys[0], ws)
    print("cold pass of", len(LAYERS), "layers, stages of", stage, flush=True)
    nnv.nnv_cold_stack(descs, kinds, raw, wt, xs, ys[1], ws, stage)
    torch.cuda.synchronize()
    for l, a, b in zip(LAYERS, *ys):
        assert torch.equal(a, b), l
        assert (b[-128:] == 7.0).all(), f"{l}: write past y"


@pytest.mark.parametrize("copies", [1, 4])
def test_launch_of_many_workgroups(env, copies):
    """Few workgroups, and more than twice what is resident at once, which take two blocks of pixels per tile: odd numbers of
    blocks, ragged last ones, every chunking mode."""
    nnv, torch = env
    layers = [Ly(64, 56, 64), Ly(96, 55, 96, 1), Ly(32, 57, 48, 5), Ly(3, 111, 64, 7, 2), Ly(20, 56, 40, 4, 1, 2), Ly(128, 33, 200, n=2, w=31)] * copies
    kinds = [nnv.IM2COL_GEMM] * len(layers)
    descs, raw, xs, wt, ws = tensors(nnv, torch, layers, kinds)
    ys = [[torch.full((l.n * l.k * l.p * l.q + 128,), 7.0, device="cuda") for l in layers] for _ in range(2)]
    one_by_one(nnv, torch, descs, kinds, raw, wt, xs, ys[0], ws)
    nnv.nnv_cold_stack(descs, kinds, raw, wt, xs, ys[1], ws, 0)
    torch.cuda.synchronize()
    for l, a, b in zip(layers, *ys):
        assert torch.equal(a, b), l
        assert (b[-128:] == 7.0).all(), f"{l}: write past y"


def build_shared(torch, how, layers, xs):
    """Inputs and outputs of a list of 32-channel 14x14 layers that share memory in the given way."""
    n = layers[0].c * layers[0].h * layers[0].w
    pool = torch.zeros(n * (len(layers) + 2), device="cuda")
    cut = lambda i, off=0: pool[i * n + off:(i + 1) * n + off]
    pool[:] = torch.cat([x for x in xs] * 2)[:pool.numel()]
    if how == "chain":
        return [cut(i) for i in range(len(layers))], [cut(i + 1) for i in range(len(layers))]
    if how == "two buffers":            # x and y change places: every layer waits for the one before
        return [cut(i % 2) for i in range(len(layers))], [cut((i + 1) % 2) for i in range(len(layers))]
    if how == "branches":               # three layers read one input, the next ones read their outputs
        return [cut(0), cut(0), cut(0), cut(2), cut(1), cut(3)], [cut(1), cut(2), cut(3), cut(4), cut(5), cut(6)]
    if how == "input written later":    # the last layers write what the first ones read
        return [cut(0), cut(1), cut(2), cut(3), cut(4), cut(5)], [cut(3), cut(4), cut(5), cut(0), cut(1), cut(2)]
    if how == "same output":            # the later layer's output stays
        return [cut(0), cut(1), cut(2), cut(0), cut(1), cut(2)], [cut(4), cut(4), cut(5), cut(5), cut(4), cut(6)]
    # outputs that start inside an earlier output or input (16-byte aligned)
    return [cut(0), cut(0, 64), cut(1), cut(2, 4), cut(0), cut(6)], [cut(1, 128), cut(3), cut(3, 64), cut(5), cut(0, 256), cut(5, 4)]


@pytest.mark.parametrize("how", ["chain", "two buffers", "branches", "input written later", "same output", "shifted"])
def test_buffers_in_common(env, how):
    nnv, torch = env
    layers = [Ly(32, 14, 32)] * 6
    kinds = [nnv.IM2COL_GEMM] * 6
    descs, raw, xs, wt, ws = tensors(nnv, torch, layers, kinds)
    got = []
    for run in range(2):
        x, y = build_shared(torch, how, layers, xs)
        pool = x[0]._base
        if run == 0:
            one_by_one(nnv, torch, descs, kinds, raw, wt, x, y, ws)
        else:
            nnv.nnv_cold_stack(descs, kinds, raw, wt, x, y, ws, 0)
        torch.cuda.synchronize()
        got.append(pool.clone())
    assert torch.equal(got[0], got[1])


def test_captured(env):
    nnv, torch = env
    kinds = [nnv.IM2COL_GEMM] * len(LAYERS)
    descs, raw, xs, wt, ws = tensors(nnv, torch, LAYERS, kinds)
    ys = [[torch.zeros(l.n * l.k * l.p * l.q, device="cuda") for l in LAYERS] for _ in range(2)]
    one_by_one(nnv, torch, descs, kinds, raw, wt, xs, ys[0], ws)
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        nnv.nnv_cold_stack(descs, kinds, raw, wt, xs, ys[1], ws, 0, stream)
    for _ in range(3):
        for y in ys[1]:
            y.zero_()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(*ys):
            assert torch.equal(a, b)
