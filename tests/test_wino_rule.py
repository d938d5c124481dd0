"""Which layers of a grouped call the library runs as the fused Winograd kernel: asked of the built library's rule (no GPU)."""
import ctypes
import os

import pytest

import paper_2206_07446_amd as nnv
from nnv_workloads import stack
from test_grouped_ranges import Geo, at

def fused(layers, kind, dtype=None, pad_w=1):
    lib = ctypes.CDLL(os.path.join(os.path.dirname(nnv.__file__), "libnnv.so"))
    rule = getattr(lib, "_ZN3nnv17wino_fused_layersEiPKNS_3GeoEiPc")
    rule.restype, rule.argtypes = None, [ctypes.c_int, ctypes.POINTER(Geo), ctypes.c_int, ctypes.POINTER(ctypes.c_char)]
    geos = (Geo * len(layers))(*[Geo(l.n, l.c, l.h, l.w, l.k, 3, 3, 1, 1, 1, pad_w, 1, nnv.F32 if dtype is None else dtype, l.h, l.w + 2 * pad_w - 2, l.c, l.k, 0) for l in layers])
    out = (ctypes.c_char * len(layers))()
    rule(len(layers), geos, kind, out)
    return [l for l, f in zip(layers, out.raw) if f]


def eligible(name, n=1, h=224, w=224):
    return [l for l in at(stack(name), n, h, w) if l.r == 3 and l.stride == 1 and l.groups == 1]


# (stack, kind, images, height, width): the most input channels of a layer that runs fused, how many of them do, and of how many
CALLS = [("vgg16", nnv.WINO_F4, 1, 224, 224, 128, 5, 13), ("vgg16", nnv.WINO_F2, 1, 224, 224, 256, 8, 13), ("vgg16", nnv.WINO_F2, 1, 96, 96, 128, 5, 13),
         ("resnet18", nnv.WINO_F2, 1, 224, 224, 0, 0, 13), ("resnet18", nnv.WINO_F4, 1, 224, 224, 0, 0, 13), ("squeezenet", nnv.WINO_F2, 1, 224, 224, 64, 8, 8)]


@pytest.mark.parametrize("name,kind,n,h,w,most,count,of", CALLS)
def test_layers_of_a_call(name, kind, n, h, w, most, count, of):
    layers = eligible(name, n, h, w)
    got = fused(layers, kind)
    assert (max((l.c for l in got), default=0), len(got), len(layers)) == (most, count, of)


def test_what_the_rule_never_takes():
    layers = eligible("vgg16")
    assert not fused(layers, nnv.WINO_F6) and not fused(layers, nnv.WINO_F4, nnv.F16)
    # patches read element by element: a longer chunk, so no more layers than with one column of padding
    assert len(fused(layers, nnv.WINO_F4, pad_w=0)) <= len(fused(layers, nnv.WINO_F4))
