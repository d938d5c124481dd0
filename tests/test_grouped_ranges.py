"""How finely a grouped call cuts the reductions of its float32 layers, read off the workspace that it asks for (no GPU)."""
import ctypes
import os
from dataclasses import replace

import pytest

import paper_2206_07446_amd as nnv
from nnv_workloads import stack
from test_gpu_split_reduction import FULL, LAYERS


class Geo(ctypes.Structure):
    """The library's own description of a layer."""
    _fields_ = [(f, ctypes.c_int) for f in "n c h w k r s sh sw ph pw groups dtype p q cg kg relu".split()]


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


# The layers of the GPU test of two-step sums that fill their tiles have the ranges (more than twelve) that it needs.
@pytest.mark.parametrize("name", list(FULL))
def test_many_ranges(name):
    half = name.startswith("f16")
    layers = LAYERS[name]
    lib = ctypes.CDLL(os.path.join(os.path.dirname(nnv.__file__), "libnnv.so"))
    ask = getattr(lib, "_ZN3nnv28im2col_items_workspace_bytesEiPKNS_3GeoEPm")
    ask.restype, ask.argtypes = None, [ctypes.c_int, ctypes.POINTER(Geo), ctypes.POINTER(ctypes.c_size_t)]
    geos = (Geo * len(layers))(*[Geo(l.n, l.c, l.h, l.w, l.k, l.r, l.s, l.stride, l.stride, l.pad, l.pad, l.groups, nnv.F16 if half else nnv.F32, l.p, l.q, l.c // l.groups, l.k // l.groups, 0)
                                     for l in layers])
    out = (ctypes.c_size_t * len(layers))()
    ask(len(layers), geos, out)
    for i, tiles, size in FULL[name]:
        l, got = layers[i], out[i]
        if half and size < 4 * 4096:        # items of single wavefronts read a copy of x
            got -= l.n * l.h * l.w * (-(-l.c // 32) * 32) * 2
        # a tile: its ranges, and 256 bytes of words of arrivals
        assert got % tiles == 0 and (got // tiles - 256) % size == 0, (l.name, got)
        print(l.name, (got // tiles - 256) // size)
        assert (got // tiles - 256) // size > 12, l.name
