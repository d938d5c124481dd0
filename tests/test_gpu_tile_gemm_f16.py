"""Float16 layers in items of whole workgroups: 3x3 and 1x1 filters at the edges of a tile, of a chunk of 32 channels, of the chunks in
flight and of a panel, alone and in a grouped call, and values that are not finite."""
import numpy as np
import pytest

from nnv_workloads import ConvLayer
from test_gpu_grouped import Case, run_grouped
from test_gpu_tile_gemm import Ly, env, forward  # noqa: F401

pytestmark = pytest.mark.gpu


def One(c, h, w, k, stride=1, pad=0, n=1):
    return ConvLayer(f"p{c}_{n}x{h}x{w}_k{k}_s{stride}p{pad}", c, h, w, k, 1, 1, stride, pad, 1, n)


def S2(c, h, w, k, pad=1, n=1):
    return ConvLayer(f"d{c}_{n}x{h}x{w}_k{k}_p{pad}", c, h, w, k, 3, 3, 2, pad, 1, n)


def Few(c, h, w, k, r, stride, pad=None, n=1):
    return ConvLayer(f"f{c}_{n}x{h}x{w}_k{k}_r{r}s{stride}", c, h, w, k, r, r, stride, r // 2 if pad is None else pad, 1, n)


# enough tiles for the path by themselves; from the sixth on 128 x 112 outputs, but for 100 channels at 57x83, whose tiles hold 64 pixels
SINGLE = [
    Ly(48, 150, 150, 64), Ly(49, 113, 200, 65, pad=0), Ly(63, 40, 41, 127, pad=2, n=6), Ly(96, 9, 9, 130, n=70), Ly(70, 1, 300, 500, n=10),
    Ly(64, 56, 56, 256, n=6), Ly(100, 57, 83, 250, n=3), Ly(33 * 2, 28, 28, 512, n=7),
    Ly(49, 41, 54, 245, n=5), Ly(100, 27, 41, 375, pad=0, n=7),
]


def check(torch, case, got):
    l = case.layer
    x, w = case.xd.cpu().double(), torch.from_numpy(case.w).half().double()
    ref = torch.nn.functional.conv2d(x, w, None if case.bd is None else case.bd.cpu().double(), stride=l.stride, padding=l.pad, groups=l.groups).clamp(min=0).numpy()
    # float16 products are exact in float32; roundings: one of 2^-24 per 32 products (and per range) of a partial sum that is at most the sum of
    # |x w|, bounded by the largest of them, and one of 2^-11 of the output
    most = float(x.abs().max()) * float(w.abs().flatten(1).sum(1).max()) + (0 if case.bd is None else float(case.bd.abs().max()))
    bound = 2.0 ** -11 * np.abs(ref) + 2.0 ** -24 * (l.c * l.r * l.s / 16 + 64) * most
    over = float((np.abs(got - ref) - bound).max())
    assert over <= 0, f"{l.name}: {over:.3e}"


@pytest.mark.parametrize("layer", SINGLE, ids=[l.name for l in SINGLE])
def test_single(env, layer):  # noqa: F811
    nnv, torch = env
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, True, 5, bias=True)
    print("case", layer, flush=True)
    need = nnv.nnv_workspace_bytes(case.desc, case.kind)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    nnv.nnv_conv_forward_relu(case.desc, case.kind, case.xd, case.wt, case.bd, case.y, ws, need)
    torch.cuda.synchronize()
    check(torch, case, case.result())


GROUPED = [
    Ly(96, 56, 56, 64), Ly(160, 28, 28, 128), Ly(224, 14, 14, 200), Ly(352, 7, 7, 512), Ly(50, 31, 57, 80, pad=2, n=3), Ly(64, 30, 1, 96),
    Ly(300, 28, 28, 90, pad=0), Ly(256, 28, 28, 256),
    # pixels in pairs (even planes) and alone (odd planes, strides, padding), ranges of whole and part of the chunks in flight
    One(256, 56, 56, 64), One(64, 56, 56, 256), One(1024, 14, 14, 256), One(255, 14, 14, 1023), One(290, 28, 28, 130, n=2), One(48, 30, 1, 600, n=5),
    One(2048, 7, 7, 512), One(512, 7, 7, 2048), One(513, 7, 9, 70, n=3), One(512, 28, 28, 1024, stride=2), One(256, 57, 55, 512, stride=2),
    One(100, 20, 21, 96, pad=1), One(70, 33, 35, 40, stride=3), One(128, 28, 28, 33, stride=2, pad=2),
    # stride 2, few channels
    S2(64, 56, 56, 128), S2(48, 57, 30, 64, pad=0), S2(200, 15, 14, 40, pad=2, n=3), S2(512, 7, 7, 512),
    Few(3, 224, 224, 64, 7, 2), Few(3, 61, 50, 32, 3, 2, n=2), Few(8, 33, 40, 70, 5, 1), Few(1, 28, 28, 6, 5, 1), Few(4, 63, 63, 96, 7, 4, pad=2), Few(3, 40, 20, 64, 3, 1),
    # beside layers that keep the other items
    One(32, 28, 28, 64), One(64, 14, 14, 24), One(3, 40, 40, 64), ConvLayer("r5", 48, 14, 14, 64, 5, 5, 1, 2), S2(32, 28, 28, 64),
    ConvLayer("s3", 64, 29, 29, 64, 3, 3, 3, 1), ConvLayer("g2", 128, 14, 14, 96, 3, 3, 1, 1, 2),
]


@pytest.mark.parametrize("count", [len(GROUPED), 22, 8])
def test_grouped(env, count):  # noqa: F811
    nnv, torch = env
    cases = [Case(nnv, torch, l, nnv.IM2COL_GEMM, True, 60 + i, bias=i % 2 == 0) for i, l in enumerate(GROUPED[:count])]
    run_grouped(nnv, torch, cases, relu=True)
    for c in cases:
        check(torch, c, c.result())


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 65504.0, 6e-8])
def test_values(env, value):  # noqa: F811
    """Infinite, NaN, the largest and the smallest float16 at the corners of a tile and of a chunk: they reach the outputs whose
    window holds them, and no other."""
    nnv, torch = env
    cases = [Case(nnv, torch, l, nnv.IM2COL_GEMM, True, 90 + i) for i, l in enumerate(GROUPED)]
    for c in cases:
        l = c.layer
        for ch, p, q in ((0, 0, 0), (l.c - 1, l.h - 1, l.w - 1), (min(31, l.c - 1), l.h // 2, 0)):
            c.x[0, ch, p, q] = value
        c.xd = torch.from_numpy(c.x).to("cuda").half()
    descs, kinds = [c.desc for c in cases], [c.kind for c in cases]
    need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    nnv.nnv_conv_forward_grouped(descs, kinds, [c.xd for c in cases], [c.wt for c in cases], None, [c.y for c in cases], ws, need, 0)
    torch.cuda.synchronize()
    for c in cases:
        l, got = c.layer, c.result()
        x = c.xd.cpu().double()
        w = torch.from_numpy(c.w).half().double()
        # (which outputs meet it: those whose window holds the pixel and whose weight there is not zero)
        clean = torch.where(torch.isfinite(x), x, torch.zeros_like(x))
        ref = torch.nn.functional.conv2d(clean, w, stride=l.stride, padding=l.pad, groups=l.groups).numpy()
        most = float(clean.abs().max()) * float(w.abs().flatten(1).sum(1).max())
        bad = torch.nn.functional.conv2d((~torch.isfinite(x)).double(), torch.ones_like(w), stride=l.stride, padding=l.pad, groups=l.groups).numpy() > 0
        tol = 2.0 ** -11 * np.abs(ref) + 2.0 ** -24 * (l.c * l.r * l.s / 16 + 64) * most + 2.0 ** -25
        with np.errstate(invalid="ignore"):
            ok = (np.abs(got - ref) <= tol) | (np.abs(ref) > 65000)
        assert ok[~bad].all(), l.name
        assert not np.isfinite(got[bad]).any(), l.name


@pytest.mark.parametrize("layer", [One(256, 56, 56, 256, n=8), Ly(64, 56, 56, 512, n=4), S2(64, 112, 112, 256, n=4), Few(3, 224, 224, 64, 7, 2)],
                         ids=["1x1", "3x3", "stride2", "few"])
def test_one_layer_grouped(env, layer):  # noqa: F811
    nnv, torch = env
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, True, 31, bias=True)
    run_grouped(nnv, torch, [case], relu=True)
    check(torch, case, case.result())
