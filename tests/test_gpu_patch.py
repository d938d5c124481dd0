"""Float32 3x3 layers whose pixels go through LDS (deep layers on small planes), and the same layers in launches of a cold pass: rows of one to many pixels, tiles that
cross rows and images, ragged channels, panels and last tiles, any number of padding rows."""
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


# (images, channels, height, width, outputs, groups, padding rows): wavefronts of 12 blocks of 4 channels (the fewest), of 13 with a ragged last one, of many
SHAPES = [(1, 768, 1, 1, 16, 1, 1), (1, 775, 4, 4, 33, 1, 1), (3, 390, 7, 7, 160, 1, 1), (2, 512, 5, 17, 100, 1, 0), (1, 1030, 3, 2, 20, 1, 2), (5, 385, 9, 1, 70, 1, 1),
          (1, 512, 7, 7, 512, 1, 1), (2, 770, 16, 14, 154, 1, 1), (1, 830, 2, 33, 48, 2, 1), (16, 800, 1, 15, 40, 1, 1), (1, 900, 20, 16, 17, 1, 1), (4, 400, 12, 31, 30, 1, 3)]


def build(nnv, torch, shape, seed):
    n, c, h, w, k, groups, ph = shape
    layer = ConvLayer("l", c, h, w, k, 3, 3, 1, 1, groups, n)
    wr, x = layer_tensors(layer, seed)
    desc = nnv.make_desc(layer, nnv.F32)
    desc.pad_h = ph
    p = h + 2 * ph - 2
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wr).double(), None, padding=(ph, 1), groups=groups)
    mag = torch.nn.functional.conv2d(torch.from_numpy(x).double().abs(), torch.from_numpy(wr).double().abs(), None, padding=(ph, 1), groups=groups)
    return desc, torch.from_numpy(wr).cuda(), torch.from_numpy(x).cuda(), ref, mag, torch.full((n * k * p * w + 128,), 7.0, device="cuda")


def test_layers(env):
    nnv, torch = env
    cases = [build(nnv, torch, s, 40 + i) for i, s in enumerate(SHAPES) if s[2] + 2 * s[6] >= 3]
    kinds = [nnv.IM2COL_GEMM] * len(cases)
    wts = [torch.empty(nnv.nnv_transformed_bytes(c[0], k), dtype=torch.uint8, device="cuda") for c, k in zip(cases, kinds)]
    for (desc, raw, x, ref, mag, y), wt in zip(cases, wts):
        print("layer", list(x.shape), list(ref.shape), flush=True)
        nnv.nnv_transform_weights(desc, nnv.IM2COL_GEMM, raw, wt)
        nnv.nnv_conv_forward(desc, nnv.IM2COL_GEMM, x, wt, None, y, None, 0)
        torch.cuda.synchronize()
        assert (y[-128:] == 7.0).all(), "write past y"
        got = y[:-128].cpu().double().reshape(ref.shape)
        # a product and a sum each round by at most 2^-24 of a partial sum of |x w|; a random walk of them, eight times over
        terms = raw[0].numel()
        assert ((got - ref).abs() <= 2.0 ** -24 * 8 * np.sqrt(terms) * mag).all(), list(ref.shape)
    ys = [torch.full_like(c[5], 7.0) for c in cases]
    nnv.nnv_cold_stack([c[0] for c in cases], kinds, [c[1] for c in cases], wts, [c[2] for c in cases], ys, None, 0)
    torch.cuda.synchronize()
    for c, y in zip(cases, ys):
        assert torch.equal(c[5], y), list(c[3].shape)
