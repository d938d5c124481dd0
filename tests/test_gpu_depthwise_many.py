"""Depthwise layers of a grouped call: columns of outputs that end inside and outside a plane, either filter, stride, storage type and
layout of the filters, pads wider than the plane."""
import pytest

from nnv_workloads import ConvLayer
from test_gpu_grouped import Case
from test_gpu_tile_gemm import env  # noqa: F401

pytestmark = pytest.mark.gpu


def Dw(c, h, w, r, stride, pad=None, n=1):
    return ConvLayer(f"d{c}_{n}x{h}x{w}_r{r}s{stride}", c, h, w, c, r, r, stride, r // 2 if pad is None else pad, c, n)


LAYERS = [Dw(c, h, w, r, s, n=n) for r in (3, 5) for s in (1, 2) for c, h, w, n in ((33, 7, 7, 1), (64, 14, 14, 2), (5, 5, 61, 3), (1, 9, 8, 1), (96, 31, 1, 1), (40, 12, 200, 1))]
LAYERS += [Dw(32, 1, 1, 3, 1, 4), Dw(7, 3, 2, 5, 2, 5, n=5), Dw(130, 6, 6, 3, 1, 0), Dw(20, 8, 5, 5, 1, 0)]


# beside them: items of single wavefronts (numbers that fill no workgroup) and, from the fourth on, of workgroups
BESIDE = [ConvLayer("a", 20, 9, 9, 24, 1, 1, 1, 0), ConvLayer("b", 300, 7, 7, 70, 1, 1, 1, 0), ConvLayer("c", 24, 13, 5, 40, 3, 3, 1, 1), ConvLayer("d", 16, 5, 5, 100, 5, 5, 1, 2)]
BESIDE += [ConvLayer(f"t{i}", 128, 56, 56, 128, 3, 3, 1, 1) for i in range(6)]


@pytest.mark.parametrize("beside", [0, 4, 10])
@pytest.mark.parametrize("kind", ["DEPTHWISE", "DIRECT"])
@pytest.mark.parametrize("half", [False, True], ids=["f32", "f16"])
def test_columns(env, kind, half, beside):  # noqa: F811
    nnv, torch = env
    cases = [Case(nnv, torch, l, getattr(nnv, kind), half, 500 + i, bias=i % 3 > 0) for i, l in enumerate(LAYERS)]
    cases += [Case(nnv, torch, l, nnv.IM2COL_GEMM, half, 540 + i, bias=i % 2 > 0) for i, l in enumerate(BESIDE[:beside])]
    descs, kinds = [c.desc for c in cases], [c.kind for c in cases]
    print("grouped call:", kind, half, [c.layer.name for c in cases], flush=True)
    need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    nnv.nnv_conv_forward_grouped(descs, kinds, [c.xd for c in cases], [c.wt for c in cases], [c.bd for c in cases], [c.y for c in cases], ws, need, nnv.FORWARD_RELU)
    torch.cuda.synchronize()
    for c in cases:
        l = c.layer
        w = torch.from_numpy(c.w)
        w = w.half().double() if half and c.kind != nnv.DIRECT else w.double()
        x = c.xd.cpu().double()
        ref = torch.nn.functional.conv2d(x, w, None if c.bd is None else c.bd.cpu().double(), stride=l.stride, padding=l.pad, groups=l.groups).clamp(min=0).numpy()
        # a chain of at most c r s / groups float32 roundings of sums below the sum of |x w| and |b|; float16: one more of the output
        most = float(x.abs().max()) * float(w.abs().flatten(1).sum(1).max()) + (0 if c.bd is None else float(c.bd.abs().max()))
        bound = (l.c // l.groups * l.r * l.s + 1) * 2.0 ** -24 * most + (2.0 ** -11 * abs(ref) + 2.0 ** -25 if half else 0)
        assert (abs(c.result() - ref) <= bound).all(), l.name
