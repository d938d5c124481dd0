"""Float32 Winograd layers whose three steps run as one kernel: the same sums, bit for bit, whichever form of it a call takes - wavefronts of their own, workgroups of one,
two or four panels and of one or two blocks of tiles, alone or in a launch with others."""
import pytest

from nnv_testlib import conv_tolerance
from nnv_workloads import ConvLayer
from test_wino_rule import fused

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2206_07446_amd as nnv
    assert torch.cuda.is_available(), "GPU tests need the HIP device"
    nnv.load()
    return nnv, torch


class Case:
    """A layer (images, channels, height, width, outputs, padding rows, padding columns), its tensors and its workspace-free or single-call output."""

    def __init__(self, nnv, torch, kind, shape, seed):
        n, c, h, w, k, ph, pw = shape
        gen = torch.Generator(device="cuda").manual_seed(seed)
        self.shape, self.kind = shape, kind
        self.desc = nnv.make_desc(ConvLayer("l", c, h, w, k, 3, 3, 1, 1, 1, n), nnv.F32)
        self.desc.pad_h, self.desc.pad_w = ph, pw
        self.raw = torch.randn((k, c, 3, 3), device="cuda", generator=gen) * (2.0 / (9 * c)) ** 0.5
        self.x = torch.rand((n, c, h, w), device="cuda", generator=gen) * 2 - 1
        self.bias = torch.randn((k,), device="cuda", generator=gen)
        self.wt = torch.empty(nnv.nnv_transformed_bytes(self.desc, kind), dtype=torch.uint8, device="cuda")
        nnv.nnv_transform_weights(self.desc, kind, self.raw, self.wt)
        self.size = n * k * (h + 2 * ph - 2) * (w + 2 * pw - 2)

    def out(self, torch):
        return torch.full((self.size + 128,), 7.0, device="cuda")


def alone(nnv, torch, case):
    print("alone", case.shape, flush=True)
    y = case.out(torch)
    ws = torch.empty(max(nnv.nnv_workspace_bytes(case.desc, case.kind), 256), dtype=torch.uint8, device="cuda")
    nnv.nnv_conv_forward(case.desc, case.kind, case.x, case.wt, case.bias, y, ws)
    torch.cuda.synchronize()
    assert (y[-128:] == 7.0).all(), "write past y"
    return y[:-128]


def together(nnv, torch, cases):
    print("together", [c.shape for c in cases], flush=True)
    descs, kinds = [c.desc for c in cases], [c.kind for c in cases]
    ws = torch.empty(max(nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds), 256), dtype=torch.uint8, device="cuda")
    ys = [c.out(torch) for c in cases]
    nnv.nnv_conv_forward_grouped(descs, kinds, [c.x for c in cases], [c.wt for c in cases], [c.bias for c in cases], ys, ws)
    torch.cuda.synchronize()
    assert all((y[-128:] == 7.0).all() for y in ys), "write past y"
    return [y[:-128] for y in ys]


# one step of channels, full and not; two, one of them ragged; more; one to eight panels of outputs, ragged ones; few workgroups and many; paddings
FEW = [(1, 3, 112, 112, 64, 1, 1), (1, 4, 112, 112, 128, 1, 1), (1, 1, 150, 97, 33, 1, 1), (2, 2, 120, 70, 96, 1, 1), (1, 3, 224, 224, 16, 1, 1), (1, 4, 300, 130, 9, 1, 1), (4, 4, 112, 112, 70, 1, 1),
       (1, 3, 140, 150, 40, 1, 0), (1, 3, 140, 150, 40, 0, 2), (8, 7, 31, 74, 38, 1, 1), (1, 6, 200, 90, 48, 1, 1), (1, 8, 56, 56, 128, 1, 1), (5, 13, 106, 7, 33, 1, 1), (2, 11, 60, 97, 20, 1, 1), (1, 30, 100, 101, 48, 1, 1)]


@pytest.mark.parametrize("kind", ["wino_f2", "wino_f4"])
def test_few_channels(env, kind):
    nnv, torch = env
    kind = nnv.KINDS[kind]
    cases = [Case(nnv, torch, kind, s, 60 + i) for i, s in enumerate(FEW)]
    cases = [c for c in cases if nnv.nnv_workspace_bytes(c.desc, kind) == 0]        # (the others have a second route)
    assert len(cases) >= 11
    for c, y in zip(cases, together(nnv, torch, cases)):
        n, _, h, w, k, ph, pw = c.shape
        ref = torch.nn.functional.conv2d(c.x.double().cpu(), c.raw.double().cpu(), c.bias.double().cpu(), padding=(ph, pw)).flatten()
        assert (y.double().cpu() - ref).abs().max() <= conv_tolerance(kind, False) * ref.abs().max(), c.shape
        assert torch.equal(alone(nnv, torch, c), y), c.shape


# layers that read their patches in wide loads (one column of padding) in a launch with layers that read them element by element
@pytest.mark.parametrize("kind", ["wino_f2", "wino_f4"])
def test_mixed_paddings(env, kind):
    nnv, torch = env
    kind = nnv.KINDS[kind]
    shapes = [(1, 16, 120, 130, 64, 1, 1), (1, 16, 120, 130, 64, 1, 0), (2, 21, 90, 101, 33, 1, 2), (2, 21, 90, 101, 33, 1, 1), (1, 40, 150, 97, 16, 0, 1), (1, 3, 130, 140, 40, 1, 0), (1, 12, 33, 64, 48, 1, 1)]
    cases = [Case(nnv, torch, kind, s, 90 + i) for i, s in enumerate(shapes)]
    mixed = together(nnv, torch, cases)
    for sort in ([c for c in cases if c.shape[6] == 1], [c for c in cases if c.shape[6] != 1]):
        for c, y in zip(sort, together(nnv, torch, sort)):
            assert torch.equal(mixed[cases.index(c)], y), c.shape
    # ... and what an unpadded layer reads where a padded one reads zeros
    n, c, h, w, k, ph, _ = shapes[0]
    carried = Case(nnv, torch, kind, (n, c, h, w + 2, k, ph, 0), 90)
    carried.x, carried.wt, carried.bias = torch.nn.functional.pad(cases[0].x, (1, 1)).contiguous(), cases[0].wt, cases[0].bias
    assert torch.equal(together(nnv, torch, [carried] + cases[1:])[0], mixed[0])


# (images, channels, height, width, outputs): ragged everything, up to 31 channel steps, which no route splits
EITHER = [(1, 64, 56, 56, 64), (2, 20, 40, 37, 70), (1, 100, 33, 40, 33), (3, 37, 21, 30, 48), (1, 124, 28, 28, 96), (2, 80, 14, 20, 130), (1, 9, 60, 61, 200), (4, 50, 14, 14, 64),
          (1, 64, 28, 28, 64), (2, 33, 30, 50, 17), (1, 120, 40, 44, 128), (5, 30, 10, 11, 40)]
# ... in three launches beside layers of many channels on few tiles, in the fused kernel beside layers of many tiles
BESIDE = {"three": [(1, 512, 14, 14, 512)] * 8, "fused": [(4, 60, 112, 112, 64), (2, 64, 150, 140, 64), (4, 96, 90, 90, 128)]}


@pytest.mark.parametrize("kind", ["wino_f2", "wino_f4"])
def test_both_routes(env, kind):
    nnv, torch = env
    kind = nnv.KINDS[kind]
    cases = [Case(nnv, torch, kind, s + (1, 1), 120 + i) for i, s in enumerate(EITHER)]
    got, takes = {}, {}
    for route, others in BESIDE.items():
        beside = [Case(nnv, torch, kind, s + (1, 1), 150 + i) for i, s in enumerate(others)]
        got[route], takes[route] = [], []
        for at in range(0, len(EITHER), 4):
            part = EITHER[at:at + 4]
            layers = [ConvLayer(str(i), c, h, w, k, 3, 3, 1, 1, 1, n) for i, (n, c, h, w, k) in enumerate(others + part)]
            names = [l.name for l in fused(layers, kind)]
            takes[route] += [str(len(others) + i) in names for i in range(len(part))]
            got[route] += together(nnv, torch, beside + cases[at:at + 4])[len(others):]
    differ = [i for i in range(len(EITHER)) if takes["fused"][i] and not takes["three"][i]]
    assert len(differ) >= 6
    for i, c in enumerate(cases):
        n, _, h, w, k, ph, pw = c.shape
        ref = torch.nn.functional.conv2d(c.x.double().cpu(), c.raw.double().cpu(), c.bias.double().cpu(), padding=(ph, pw)).flatten()
        assert (got["three"][i].double().cpu() - ref).abs().max() <= conv_tolerance(kind, False) * ref.abs().max(), c.shape
        assert torch.equal(got["three"][i], got["fused"][i]), (c.shape, i in differ)
        assert torch.equal(alone(nnv, torch, c), got["fused"][i]), c.shape
