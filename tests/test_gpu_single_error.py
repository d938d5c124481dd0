"""Float32 3x3 layers in calls of their own: how far their sums may be from the exact ones."""
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


def chains(cols, wts, parts):
    """cols [steps, 4, pixels], wts [steps, 4, outputs] in float64: the sums over steps and channels as `parts` chains of float32 multiply-adds,
    added one after the other in float32."""
    steps = cols.shape[0]
    per = -(-steps // parts)
    out = np.zeros((wts.shape[2], cols.shape[2]), np.float32)
    for p in range(0, steps, per):
        acc = np.zeros_like(out)
        for s in range(p, min(p + per, steps)):
            for c in range(4):
                acc = (acc.astype(np.float64) + np.outer(wts[s, c], cols[s, c])).astype(np.float32)
        out += acc
    return out


# (channels, height and width, outputs, stride, chains): one chain for each of the wavefronts that 2048 of them leave a tile of two panels
@pytest.mark.parametrize("c,hw,k,stride,parts", [(64, 56, 64, 1, 8), (128, 28, 128, 1, 16), (64, 56, 128, 2, 16), (100, 40, 96, 1, 8)])
def test_error_of_a_layer(env, c, hw, k, stride, parts):
    nnv, torch = env
    layer = ConvLayer("l", c, hw, hw, k, 3, 3, stride, 1)
    w, x = layer_tensors(layer, 50 + c)
    desc = nnv.make_desc(layer, nnv.F32)
    raw, xd = torch.from_numpy(w).cuda(), torch.from_numpy(x).cuda()
    wt = torch.empty(nnv.nnv_transformed_bytes(desc, nnv.IM2COL_GEMM), dtype=torch.uint8, device="cuda")
    y = torch.empty((k, layer.p * layer.q), device="cuda")
    nnv.nnv_transform_weights(desc, nnv.IM2COL_GEMM, raw, wt)
    nnv.nnv_conv_forward(desc, nnv.IM2COL_GEMM, xd, wt, None, y, None, 0)
    torch.cuda.synchronize()
    # [blocks of 4 channels][taps][channels of a block]
    cols = torch.nn.functional.unfold(torch.from_numpy(x).double().reshape(1, c, hw, hw), 3, padding=1, stride=stride)[0].numpy()
    cols = cols.reshape(c // 4, 4, 9, -1).transpose(0, 2, 1, 3).reshape(c // 4 * 9, 4, -1)
    wts = w.astype(np.float64).reshape(k, c // 4, 4, 9).transpose(1, 3, 2, 0).reshape(c // 4 * 9, 4, k)
    exact = np.einsum("scp,sck->kp", cols, wts, optimize=True)
    far = lambda v: np.linalg.norm(v - exact) / np.linalg.norm(exact)       # noqa: E731
    model, got = far(chains(cols, wts, parts)), far(y.cpu().numpy().astype(np.float64))
    print(f"c={c} hw={hw} k={k} stride={stride}: {got:.3e}, {parts} chains {model:.3e}", flush=True)
    # (tens of thousands of outputs: the norms of equally long chains agree to a few per cent; chains twice as long are 1.3 times as far)
    assert got <= 1.1 * model
