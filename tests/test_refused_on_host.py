"""Layers that the library refuses when asked to run them, seen without a GPU: no launch is tried."""
import ctypes
import os

import pytest
import torch

import paper_2206_07446_amd as nnv
from nnv_workloads import ConvLayer

# (the pointers below are no memory: a call that is not refused must find no GPU)
pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="passes addresses that are not memory; runs where there is no GPU to use them")


def call(fn, *args):
    lib = ctypes.CDLL(os.path.join(os.path.dirname(nnv.__file__), "libnnv.so"))
    lib.nnv_last_hip_error.restype = ctypes.c_char_p
    rc = getattr(lib, fn)(*args)
    return rc, lib.nnv_last_hip_error().decode()


def test_winograd_of_too_many_tiles():
    # 12 001 padded zeros around one pixel: 36 million tiles of F(2x2), more than 65535 x 16 blocks of 16
    desc = nnv.make_desc(ConvLayer("l", 1, 1, 1, 1, 3, 3, 1, 6001), nnv.F32)
    assert nnv.nnv_kind_supported(desc, nnv.WINO_F2) == 1 and nnv.nnv_workspace_bytes(desc, nnv.WINO_F2) == 0
    x, w, y = (ctypes.c_void_p(v << 40) for v in (1, 2, 3))
    rc, text = call("nnv_conv_forward", ctypes.byref(desc), nnv.WINO_F2, x, w, None, y, None, ctypes.c_size_t(0), None)
    assert rc == -6 and text == "invalid argument"
    n = 3
    descs, kinds = (type(desc) * n)(*[desc] * n), (ctypes.c_int * n)(*[nnv.WINO_F2] * n)
    xs, ws, ys = ((ctypes.c_void_p * n)(*[(v * 16 + i) << 40 for i in range(n)]) for v in (1, 2, 3))
    need = nnv.nnv_conv_forward_grouped_workspace_bytes([desc] * n, [nnv.WINO_F2] * n)
    rc, text = call("nnv_conv_forward_grouped", n, descs, kinds, xs, ws, None, ys, ctypes.c_void_p(4 << 40), ctypes.c_size_t(need), 0, None)
    assert rc == -6 and text == "invalid argument"
