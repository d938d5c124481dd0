"""Reductions cut into ranges whose partial sums meet in the workspace: the last item of a tile adds them, whatever the workspace held
before, call after call and in replays of a graph."""
import pytest

from nnv_workloads import ConvLayer
from test_gpu_grouped import Case, PAD
from test_gpu_tile_gemm import env  # noqa: F401
from test_gpu_tile_gemm_f16 import check as check_f16

pytestmark = pytest.mark.gpu


def Ly(c, h, k, r=3, stride=1, n=1, w=None, groups=1):
    return ConvLayer(f"s{c}_{n}x{h}x{w or h}_k{k}_r{r}s{stride}g{groups}", c, h, w or h, k, r, r, stride, r // 2, groups, n)


# two ranges and as many as the channels allow, every sort of item: workgroups of 64 x 112 and 64 x 64 outputs (3x3; 1x1 in pairs of pixels and alone), wavefronts
# of one, two and four panels, ragged last panels, pixels and ranges
LAYERS = {
    "f32": [Ly(64, 56, 64), Ly(128, 28, 128), Ly(256, 14, 250), Ly(512, 7, 512), Ly(500, 14, 60), Ly(256, 14, 512, 3, 2), Ly(512, 14, 96, 1), Ly(300, 9, 16, 1),
            Ly(130, 13, 20, 3, 2), Ly(96, 14, 48, 5), Ly(20, 30, 64, 7, 2), Ly(256, 14, 96, groups=2), Ly(520, 5, 30, 1, n=3)],
    "f16": [Ly(512, 7, 512), Ly(1024, 14, 256, 1), Ly(2048, 7, 512, 1), Ly(1024, 7, 70, 1), Ly(512, 14, 512, 3, 2), Ly(512, 14, 250, n=2), Ly(2048, 8, 100, 1),
            Ly(1024, 14, 130, 1, 2), Ly(256, 14, 40, 5), Ly(1152, 7, 24, 1), Ly(320, 3, 20, 1), Ly(768, 4, 48)],
}

# ranges in groups (more than twelve of them): wavefronts of 4, 2 and 1 panels, the last group a single range or short; workgroups
LAYERS["f32 groups"] = [Ly(512, 5, 512, w=4), Ly(1024, 4, 40), Ly(700, 3, 16), Ly(400, 6, 130, 5), Ly(1000, 4, 64, 1), Ly(512, 4, 24, 3, 2), Ly(470, 2, 80)]
LAYERS["f32 groups, workgroups"] = [Ly(1100, 14, 128), Ly(900, 7, 100, n=4), Ly(64, 20, 64), Ly(832, 8, 70)] * 2
LAYERS["f16 groups"] = [Ly(3072, 4, 16, w=8), Ly(3000, 8, 32, w=4), Ly(2048, 3, 16), Ly(2048, 2, 40), Ly(1500, 3, 24, 5), Ly(2000, 3, 20, 1)]
LAYERS["f16 groups, workgroups"] = [Ly(2048, 8, 256, n=2, w=14), Ly(2048, 16, 64, 3, 2, n=2), Ly(2000, 8, 64, w=14), Ly(2048, 7, 100, n=2), Ly(1900, 13, 70, 3, 2)]
# layers that fill their tiles: (index in the list, tiles, bytes of a tile's range); more than twelve ranges each (test_grouped_ranges.py counts them)
FULL = {"f32 groups": [(0, 8, 4 * 2048)], "f16 groups": [(0, 1, 2048), (1, 1, 2 * 2048)], "f16 groups, workgroups": [(0, 8, 7 * 4096), (1, 2, 4 * 4096), (2, 1, 7 * 4096)]}


@pytest.mark.parametrize("dtype", list(LAYERS))
def test_any_workspace(env, dtype):  # noqa: F811
    nnv, torch = env
    half = dtype.startswith("f16")
    # (copies of the list: float16 layers run in workgroups from some number of items on)
    layers = LAYERS[dtype] * (3 if dtype == "f16" else 1)
    cases = [Case(nnv, torch, l, nnv.IM2COL_GEMM, half, 300 + i, bias=i % 2 == 0) for i, l in enumerate(layers)]
    descs, kinds = [c.desc for c in cases], [c.kind for c in cases]
    need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
    assert need > 0
    print("grouped call:", dtype, [l.name for l in layers], flush=True)
    wsbuf = torch.zeros(need + 2 * PAD, dtype=torch.uint8, device="cuda")
    ws = wsbuf[PAD:PAD + need]

    def call(stream=None):
        nnv.nnv_conv_forward_grouped(descs, kinds, [c.xd for c in cases], [c.wt for c in cases], [c.bd for c in cases], [c.y for c in cases], ws, need,
                                     nnv.FORWARD_RELU, stream=stream)

    first = None
    for fill in ("zeros", "ones", "noise", "as the last call left it", "shifted", "words of an earlier launch"):
        if fill == "ones":
            wsbuf.fill_(255)
        elif fill == "noise":
            ws[:need // 4 * 4].view(torch.float32).normal_()
        elif fill == "shifted":             # partial sums where the words of arrivals were
            ws.copy_(torch.roll(ws.clone(), 4096 + 16))
        elif fill == "words of an earlier launch":      # the process's first one, whose workspace another call overwrote: one arrival everywhere
            ws[:need // 8 * 8].view(torch.int64).fill_(0x7fa5c3e996b1 << 16 | 1)
        wsbuf[:PAD] = 0x5A
        wsbuf[PAD + need:] = 0x5A
        for c in cases:
            c.y.fill_(0x7F)
        call()
        torch.cuda.synchronize()
        assert (wsbuf[:PAD] == 0x5A).all() and (wsbuf[PAD + need:] == 0x5A).all(), "write outside the workspace"
        if first is None:
            first = [c.ybuf.clone() for c in cases]
            for c in cases:
                if half:
                    check_f16(torch, c, c.result())
                else:
                    l = c.layer
                    ref = torch.nn.functional.conv2d(c.xd.cpu().double(), torch.from_numpy(c.w).double(), None if c.bd is None else c.bd.cpu().double(), stride=l.stride,
                                                     padding=l.pad, groups=l.groups).clamp(min=0).numpy()
                    # every sum of the chain rounds by at most 2^-24 of the sum of |x w|, which |x| <= 1 and He-normal weights keep below the bound here
                    most = float(torch.from_numpy(c.w).abs().flatten(1).sum(1).max()) + 1
                    bound = 2.0 ** -24 * (l.c // l.groups * l.r * l.s / 4 + 64) * most
                    assert abs(c.result() - ref).max() <= bound, l.name
        for c, f in zip(cases, first):
            assert torch.equal(c.ybuf, f), (fill, c.layer.name)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(side)
    for i in range(3):
        for c in cases:
            c.y.fill_(0x7F)
        if i == 1:
            ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        for c, f in zip(cases, first):
            assert torch.equal(c.ybuf, f), ("replay", i, c.layer.name)
