"""Float32 3x3 layers in items of whole workgroups (three bfloat16 parts per float32): sizes at the edges of a tile, of a
chunk of 32 channels and of a panel, alone and in a grouped call, and values that bfloat16 cannot hold."""
import numpy as np
import pytest

from nnv_workloads import ConvLayer, layer_tensors
from oracle import cdirect
from test_gpu_grouped import Case, run_grouped

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2206_07446_amd as nnv
    assert torch.cuda.is_available(), "GPU tests need the HIP device"
    nnv.load()
    return nnv, torch


def Ly(c, h, w, k, pad=1, n=1):
    return ConvLayer(f"c{c}_{n}x{h}x{w}_k{k}_p{pad}", c, h, w, k, 3, 3, 1, pad, 1, n)


def forward(nnv, torch, case, relu=False):
    (nnv.nnv_conv_forward_relu if relu else nnv.nnv_conv_forward)(case.desc, case.kind, case.xd, case.wt, case.bd, case.y, None, 0)
    torch.cuda.synchronize()
    return case.result()


# at least 200 items of 64 x 112 outputs or 350 of 64 x 64: such layers take the path by themselves (65 channels at 110 x 7x7 stay just below)
SINGLE = [
    Ly(48, 150, 150, 64), Ly(49, 113, 200, 65, pad=0), Ly(64, 58, 61, 400, n=2), Ly(63, 40, 41, 127, pad=2, n=6),
    Ly(96, 9, 9, 130, n=70), Ly(65, 7, 7, 128, n=110), Ly(128, 224, 113, 33), Ly(70, 1, 300, 500, n=10),
    Ly(65, 7, 7, 128, n=180), Ly(64, 56, 56, 256, n=6), Ly(100, 57, 83, 250, n=3),
    # 128 x 112 outputs with two buffers: at most 512 items, where 64 x 112 would be more than 768
    Ly(64, 56, 56, 256, n=8), Ly(49, 41, 54, 245, n=11), Ly(70, 41, 54, 249, n=10),
]


@pytest.mark.parametrize("layer", SINGLE, ids=[l.name for l in SINGLE])
def test_single(env, layer):
    nnv, torch = env
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, False, 5, bias=True)
    print("case", layer, flush=True)
    got = forward(nnv, torch, case, relu=True)
    ref = case.reference(big=True)
    # the sum over 9 C products: half an ulp each time an accumulator is rounded, twice per 32 channels and tap, of a partial sum
    # that is at most sum |x w|
    bound = np.abs(cdirect.conv2d_direct_c(np.abs(case.x), np.abs(case.w), 1, layer.pad, 1)).max() * 2.0 ** -24 * 18 * -(-layer.c // 32)
    assert np.abs(got - np.maximum(ref, 0.0)).max() <= bound + 2.0 ** -23 * np.abs(ref).max()
    # a random walk of those roundings, four times over
    rel = np.linalg.norm(got - np.maximum(ref, 0.0)) / np.linalg.norm(ref)
    assert rel <= 4 * 2.0 ** -24 * np.sqrt(18 * -(-layer.c // 32)), f"{layer.name}: {rel:.2e}"


def test_grouped_ranges(env):
    """Channel counts whose ranges are unequal, tiles of both widths, ragged planes, beside layers that keep the other items."""
    nnv, torch = env
    layers = [Ly(96, 56, 56, 64), Ly(160, 28, 28, 128), Ly(224, 14, 14, 200), Ly(352, 7, 7, 512), Ly(50, 31, 57, 80, pad=2, n=3),
              Ly(256, 20, 24, 256), Ly(64, 30, 1, 96), Ly(300, 28, 28, 90, pad=0),
              ConvLayer("s2", 64, 56, 56, 128, 3, 3, 2, 1), ConvLayer("pw", 96, 28, 28, 64, 1, 1, 1, 0), ConvLayer("stem", 3, 64, 64, 64, 7, 7, 2, 3)]
    run_grouped(nnv, torch, [Case(nnv, torch, l, nnv.IM2COL_GEMM, False, 60 + i, bias=i % 2 == 0) for i, l in enumerate(layers)])


@pytest.mark.parametrize("ks", [(64, 64, 64, 64), (64, 128, 64), (192, 64, 48)])
def test_wide_7x7(env, ks):
    """7x7 layers in a launch of one to one and a half times as many items as are resident at once: four panels per tile."""
    nnv, torch = env
    layers = [ConvLayer(f"w{i}", (3, 5, 4, 3)[i], (224, 201, 223, 224)[i], (224, 230, 225, 224)[i], k, 7, 7, 2, (3, 0, 3, 2)[i]) for i, k in enumerate(ks)]
    layers += [Ly(32, 14, 14, 64), ConvLayer("pw", 96, 14, 14, 64, 1, 1, 1, 0)]
    run_grouped(nnv, torch, [Case(nnv, torch, l, nnv.IM2COL_GEMM, False, 80 + i, bias=i % 2 == 0) for i, l in enumerate(layers)], big=True)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.395e38, 1e-38])
@pytest.mark.parametrize("grouped", [False, True])
def test_values_beyond_bfloat16(env, value, grouped):
    """Infinite, NaN, finite but rounded up to infinity by bfloat16 (times weights small enough for a finite sum), and tiny."""
    nnv, torch = env
    layer = Ly(64, 150, 150, 64)
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, False, 9)
    for pos in ((0, 0, 0, 0), (0, 63, 149, 77), (0, 31, 70, 149)):
        case.x[pos] = value
    if abs(value) < 1:
        case.x[:] = (case.x * np.float32(value)).astype(np.float32)
    scale = np.float32(1e-3) if abs(value) > 1e38 and np.isfinite(value) else np.float32(1)
    case.w = (case.w * scale).astype(np.float32)
    case.xd = torch.from_numpy(case.x).to("cuda")
    nnv.nnv_transform_weights(case.desc, case.kind, torch.from_numpy(case.w).to("cuda"), case.wt)
    if grouped:
        others = [Case(nnv, torch, Ly(64, 56, 56, 128), nnv.IM2COL_GEMM, False, 70 + i) for i in range(4)]
        all_ = [case, *others]
        descs, kinds = [c.desc for c in all_], [c.kind for c in all_]
        need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
        ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        nnv.nnv_conv_forward_grouped(descs, kinds, [c.xd for c in all_], [c.wt for c in all_], None, [c.y for c in all_], ws, need, 0)
        torch.cuda.synchronize()
        got = case.result()
    else:
        got = forward(nnv, torch, case)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = cdirect.conv2d_direct_c(case.x, case.w, 1, 1, 1)
    assert (np.isnan(got) == np.isnan(ref)).all()
    inf = np.isinf(ref)
    assert (got[inf] == ref[inf]).all()
    fin = np.isfinite(ref)
    assert np.isfinite(got[fin]).all()
    if abs(value) < 1:      # sums of subnormal products: an absolute error of a few of the smallest numbers
        assert np.abs(got - ref).max() <= 64 * 18 * 2.0 ** -149 + 1e-5 * np.abs(ref).max()
    else:
        far = fin & (np.abs(ref) < 1e30)
        assert np.abs(got[far] - ref[far]).max() <= 1e-4 * np.abs(ref[far]).max()
        near = fin & ~far
        if near.any():
            assert (np.abs(got[near] - ref[near]) <= 1e-5 * np.abs(ref[near])).all()


def run_alone_or_grouped(nnv, torch, case, grouped):
    """The case's output with its present x and w, alone or as the first of a grouped call."""
    case.xd = torch.from_numpy(case.x).to("cuda")
    nnv.nnv_transform_weights(case.desc, case.kind, torch.from_numpy(case.w).to("cuda"), case.wt)
    if not grouped:
        return forward(nnv, torch, case)
    all_ = [case, *(Case(nnv, torch, Ly(64, 56, 56, 128), nnv.IM2COL_GEMM, False, 70 + i) for i in range(4))]
    descs, kinds = [c.desc for c in all_], [c.kind for c in all_]
    need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, kinds)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    nnv.nnv_conv_forward_grouped(descs, kinds, [c.xd for c in all_], [c.wt for c in all_], None, [c.y for c in all_], ws, need, 0)
    torch.cuda.synchronize()
    return case.result()


def scaled(rng, shape, exponent):
    """Magnitudes in [2^exponent, 2^(exponent + 1)], either sign."""
    return (rng.uniform(1.0, 2.0, shape) * rng.choice((-1.0, 1.0), shape) * 2.0 ** exponent).astype(np.float32)


# 128 x 112 outputs with two buffers, 64 x 112 outputs
RANGES = [Ly(64, 56, 56, 256, n=8), Ly(64, 150, 150, 64)]


@pytest.mark.parametrize("layer", RANGES, ids=[l.name for l in RANGES])
@pytest.mark.parametrize("ex,ew", [(-126, 80), (80, -126), (-140, 100), (100, -140), (-112, 60), (-75, -75), (-90, -40), (110, -100), (-100, 110), (60, 40)])
@pytest.mark.parametrize("part", [1, 2])
def test_operand_ranges(env, layer, ex, ew, part):
    """Small pixels beside large weights and the reverse, subnormal ones, products that underflow, sums that nearly overflow; in every
    channel (part 1) or in every second one beside ordinary values of about the same product (part 2)."""
    nnv, torch = env
    rng = np.random.default_rng(1000 + ex)
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, False, 5)
    case.x, case.w = scaled(rng, case.x.shape, ex), scaled(rng, case.w.shape, ew)
    if part == 2:
        case.x[:, ::2] = scaled(rng, case.x[:, ::2].shape, (ex + ew) // 2)
        case.w[:, ::2] = scaled(rng, case.w[:, ::2].shape, ex + ew - (ex + ew) // 2)
    got = run_alone_or_grouped(nnv, torch, case, part == 2 and layer.n == 1)
    ref = cdirect.conv2d_direct_c(case.x, case.w, 1, layer.pad, 1)
    # as test_single, and half of the smallest number where the result is subnormal; products are rounded to it in float32
    chunks = -(-layer.c // 32)
    err = np.linalg.norm(got - ref)
    assert err <= 4 * 2.0 ** -24 * np.sqrt(18 * chunks) * np.linalg.norm(ref) + 2.0 ** -149 * np.sqrt(ref.size), f"{err / np.linalg.norm(ref):.2e}"


@pytest.mark.parametrize("grouped", [False, True])
def test_single_products(env, grouped):
    """Outputs of one product each, all others being zero: no less exact than a float32 product."""
    nnv, torch = env
    layer = Ly(64, 150, 150, 64)
    rng = np.random.default_rng(77)
    case = Case(nnv, torch, layer, nnv.IM2COL_GEMM, False, 5)
    case.x = scaled(rng, case.x.shape, 0)
    w = scaled(rng, case.w.shape, 0)
    case.w = np.zeros_like(w)
    for k in range(layer.k):
        c, r, s = k * 5 % 64, k % 3, k // 3 % 3
        case.w[k, c, r, s] = w[k, c, r, s]
    got = run_alone_or_grouped(nnv, torch, case, grouped)
    ref = cdirect.conv2d_direct_c(case.x, case.w, 1, 1, 1)
    # half an ulp of the result, and a few roundings of its part below 2^-8
    bound = 2.0 ** -24 * (1 + 2.0 ** -5)
    worst = np.abs(got - ref)[ref != 0] / np.abs(ref)[ref != 0]
    assert worst.max() <= bound, f"{worst.max():.3e}"
    assert (got[ref == 0] == 0).all()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_values_in_ranges_of_channels(env, value):
    """A launch that splits the channels: the range with the value in it, and it alone, has sums that are not finite."""
    nnv, torch = env
    case = Case(nnv, torch, Ly(352, 14, 14, 512), nnv.IM2COL_GEMM, False, 9)
    case.x[0, 300, 13, 0] = case.x[0, 3, 5, 5] = value
    case.w[7] = 0.0          # nothing but products with zero: NaN
    got = run_alone_or_grouped(nnv, torch, case, True)
    with np.errstate(invalid="ignore"):
        ref = cdirect.conv2d_direct_c(case.x, case.w, 1, 1, 1)
    assert (np.isnan(got) == np.isnan(ref)).all()
    inf, fin = np.isinf(ref), np.isfinite(ref)
    assert (got[inf] == ref[inf]).all()
    assert np.abs(got[fin] - ref[fin]).max() <= 1e-4 * np.abs(ref[fin]).max()
