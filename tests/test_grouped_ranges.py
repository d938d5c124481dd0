"""How finely a grouped call cuts the reductions of its float32 layers, read off the workspace that it asks for (no GPU)."""
from dataclasses import replace

import pytest

import paper_2206_07446_amd as nnv
from nnv_workloads import stack


def at(layers, n, h, w):
    def size(v, to, r, pad):
        return v if v == 1 else max(r - 2 * pad, 1, -(-v * to // 224))
    return [replace(l, h=size(l.h, h, l.r, l.pad), w=size(l.w, w, l.s, l.pad), n=n) for l in layers]


# Calls of one to one and a half times the items that are resident at once, with so few chunks of channels that the range of a workgroup is the shortest one, two chunks
# of 32 channels.  (A longer range is a longer chain of sums, further from the exact ones.)
@pytest.mark.parametrize("name,n,h,w", [("alexnet", 2, 314, 246), ("alexnet", 3, 224, 200), ("alexnet", 4, 200, 180)])
def test_ranges_of_two_chunks(name, n, h, w):
    layers = at(stack(name), n, h, w)
    descs = [nnv.make_desc(l, nnv.F32) for l in layers]
    need = nnv.nnv_conv_forward_grouped_workspace_bytes(descs, [nnv.IM2COL_GEMM] * len(descs))
    # A layer that is cut keeps a partial sum of every output for each of its ranges: two chunks in the 3x3 layers; items of single wavefronts (5x5) take 144 steps of
    # four channels and a tap, to the nearest number of them.
    ranges = [(l, -(-l.c // 64)) for l in layers if l.r == 3] + [(l, (l.c * 25 // 4 + 72) // 144) for l in layers if l.r == 5]
    assert len(ranges) == 4
    assert need >= sum(4 * l.n * l.k * l.p * l.q * r for l, r in ranges if r > 1)
