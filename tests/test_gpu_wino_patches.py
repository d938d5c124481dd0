"""Float32 Winograd layers with one column of padding, whose patches are read in wide loads, against the same layers on inputs that carry the column themselves
(no padding along the rows), whose patches are read element by element: the same sums, bit for bit."""
import pytest

from nnv_testlib import conv_tolerance
from nnv_workloads import ConvLayer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2206_07446_amd as nnv
    assert torch.cuda.is_available(), "GPU tests need the HIP device"
    nnv.load()
    return nnv, torch


# (images, channels, height, width, outputs, padding rows): rows of one tile, of one partly outside, of 15, 16 and 17 tiles and more; rows of tiles that begin inside
# a row of lanes; images of odd sizes, whose last elements are the end of x; channels that fill no step
SHAPES = [(1, 5, 3, 1, 16, 1), (1, 8, 1, 3, 20, 1), (2, 19, 7, 7, 33, 1), (3, 6, 9, 13, 16, 1), (1, 17, 12, 31, 48, 0), (1, 4, 5, 64, 70, 1), (1, 33, 6, 67, 64, 2),
          (2, 16, 14, 35, 65, 1), (1, 7, 30, 101, 24, 1), (1, 70, 11, 130, 40, 1), (4, 64, 56, 56, 64, 1), (1, 12, 150, 149, 96, 1),
          # layers of many tiles, all three steps in one kernel: one, two and four panels of outputs and a ragged fifth, one to many chunks of channels and ragged last ones
          (1, 1, 200, 201, 9, 1), (1, 22, 180, 190, 16, 1), (1, 30, 224, 225, 24, 1), (2, 40, 150, 170, 33, 1), (1, 64, 224, 224, 64, 1), (1, 121, 223, 190, 70, 1), (5, 96, 110, 90, 130, 0)]


def forward(nnv, torch, kind, layers, grouped):
    """layers: (images, channels, height, width, outputs, padding rows, padding columns, x, w); the outputs."""
    descs, wts, ys, wss = [], [], [], []
    for n, c, h, w, k, ph, pw, x, raw in layers:
        desc = nnv.make_desc(ConvLayer("l", c, h, w, k, 3, 3, 1, 1, 1, n), nnv.F32)
        desc.pad_h, desc.pad_w = ph, pw
        wt = torch.empty(nnv.nnv_transformed_bytes(desc, kind), dtype=torch.uint8, device="cuda")
        nnv.nnv_transform_weights(desc, kind, raw, wt)
        descs.append(desc); wts.append(wt)
        ys.append(torch.full((n * k * (h + 2 * ph - 2) * (w + 2 * pw - 2) + 128,), 7.0, device="cuda"))
    kinds, xs = [kind] * len(layers), [l[7] for l in layers]
    if grouped:
        ws = torch.empty(max(nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds), 256), dtype=torch.uint8, device="cuda")
        nnv.nnv_conv_forward_grouped(descs, kinds, xs, wts, None, ys, ws)
    else:
        for d, x, wt, y in zip(descs, xs, wts, ys):
            wss.append(torch.empty(max(nnv.nnv_workspace_bytes(d, kind), 256), dtype=torch.uint8, device="cuda"))
            nnv.nnv_conv_forward(d, kind, x, wt, None, y, wss[-1])
    torch.cuda.synchronize()
    assert all((y[-128:] == 7.0).all() for y in ys), "write past y"
    return [y[:-128] for y in ys]


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("kind", ["wino_f2", "wino_f4", "wino_f6"])
def test_wide_loads(env, kind, grouped):
    nnv, torch = env
    kind = nnv.KINDS[kind]
    gen = torch.Generator(device="cuda").manual_seed(20)
    padded, carried = [], []
    for i, (n, c, h, w, k, ph) in enumerate(SHAPES):
        if h + 2 * ph < 3:
            continue
        x = torch.randn((n, c, h, w), device="cuda", generator=gen)
        if i % 3 == 2:      # what is not finite stays where it is
            x[:, c // 2, h // 2, w // 2] = float("inf")
            x[0, 0, h - 1, w - 1] = float("nan")
        raw = torch.randn((k * c * 9,), device="cuda", generator=gen)
        padded.append((n, c, h, w, k, ph, 1, x, raw))
        carried.append((n, c, h, w + 2, k, ph, 0, torch.nn.functional.pad(x, (1, 1)).contiguous(), raw))
    a, b = forward(nnv, torch, kind, padded, grouped), forward(nnv, torch, kind, carried, grouped)
    for l, u, v in zip(padded, a, b):
        n, c, h, w, k, ph = l[:6]
        ref = torch.nn.functional.conv2d(l[7].double().cpu(), l[8].double().cpu().reshape(k, c, 3, 3), None, padding=(ph, 1)).flatten()
        ok = torch.isfinite(ref)
        # the bound on |y - y64| / max |y| that all tests of this library hold a kind to
        assert (u.cpu().double() - ref)[ok].abs().max() <= conv_tolerance(kind, False) * ref[ok].abs().max() or not torch.isfinite(l[7]).all(), l[:6]
        assert torch.equal(torch.nan_to_num(u, 3e38, 2e38, 1e38), torch.nan_to_num(v, 3e38, 2e38, 1e38)), l[:6]
