"""The calls a program makes per pass, through the compiled module and through ctypes: what reaches the
library and what is refused, without touching a GPU (every call but those of the last test ends at an argument check)."""
import ctypes
import sysconfig

import pytest
import torch

import paper_2206_07446_amd as nnv
from paper_2206_07446_amd import binding, build

NULL, UNSUPPORTED, WORKSPACE, ALIGN, ARG = -1, -3, -4, -5, -7


def desc(**kw):
    base = dict(n=1, c=16, h=32, w=32, k=16, r=3, s=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, groups=1, dtype=0)
    return nnv.ConvDesc(**{**base, **kw})


@pytest.fixture(params=["module", "ctypes"])
def calls(request, monkeypatch):
    nnv.load()
    if request.param == "module":
        assert binding._native.__name__ == "_nnvpy", "the compiled module is what runs here"
    else:
        monkeypatch.setattr(binding, "_native", binding._CtypesCalls)
    return binding


def status(fn, *args, **kw):
    with pytest.raises(nnv.NnvError) as e:
        fn(*args, stream=0, **kw)
    return e.value.status


A = 256     # an aligned address that is never followed


def test_single_calls(calls):
    d = desc()
    for fn in (nnv.nnv_conv_forward, nnv.nnv_conv_forward_relu):
        assert status(fn, d, 1, None, A, None, A, None) == NULL
        assert status(fn, d, 9, A, A, None, A, None) == ARG
        assert status(fn, d, 4, A, A, None, A, None) == UNSUPPORTED
        assert status(fn, d, 1, A + 4, A, None, A, None) == ALIGN
        assert status(fn, d, 1, A, A, A + 2, A, None) == ALIGN
        assert status(fn, d, 3, A, A, None, A, A, 16) == WORKSPACE
        assert status(fn, d, 3, A, A, None, A, torch.empty(64)) == WORKSPACE          # the size of the tensor
        assert status(fn, d, 3, A, A, None, A + 4, torch.empty(64), 1 << 30) == ALIGN  # an explicit size wins
        assert status(fn, d, 3, A, A, None, A, None) == NULL
    assert status(nnv.nnv_conv_forward_static, d, 1, A, None, None, A) == NULL
    assert status(nnv.nnv_conv_forward_static, desc(c=1088, k=1088, h=112, w=112), 3, A, A, None, A) == WORKSPACE
    assert status(nnv.nnv_transform_weights, d, 1, None, A) == NULL
    assert status(nnv.nnv_transform_weights, d, 1, A, A + 4) == ALIGN


def test_lists(calls):
    d, n = desc(), 3
    ds, ks, ps = [d] * n, [1] * n, [A] * n
    assert status(nnv.nnv_transform_weights_grouped, ds, ks, ps, [A, A, A + 4]) == ALIGN
    assert status(nnv.nnv_transform_weights_grouped, tuple(ds), (1, 1, 9), tuple(ps), tuple(ps)) == ARG
    f = nnv.nnv_conv_forward_grouped
    assert status(f, ds, ks, [A, None, A], ps, None, ps, None) == NULL
    assert status(f, ds, ks, ps, ps, [None, A + 2, A], ps, None) == ALIGN
    assert status(f, ds, ks, ps, ps, None, ps, None, flags=2) == ARG
    assert status(f, ds, [3] * n, ps, ps, None, ps, torch.empty(64)) == WORKSPACE
    f([], [], [], [], None, [], None, stream=0)
    for args in ((ds, ks, [A, A + 4, A], ps, ps, ps, None), (ds, ks, ps, ps, ps, [A + 4, A, A], None)):
        with pytest.raises(nnv.NnvError) as e:
            nnv.nnv_cold_stack(*args, stream_exec=0)
        assert e.value.status == ALIGN


@pytest.mark.parametrize("off", [-1, 1], ids=["short", "long"])
def test_lists_of_another_length_are_refused(calls, off):
    ds, ks, ps = [desc()] * 3, [1] * 3, [A] * 3
    wrong = [A] * (3 + off)
    for i in range(1, 4):
        args = [ds, ks, ps, ps]
        args[i] = [1] * (3 + off) if i == 1 else wrong
        with pytest.raises(ValueError):
            nnv.nnv_transform_weights_grouped(*args, stream=0)
    for i in range(1, 6):
        args = [ds, ks, ps, ps, ps, ps]
        args[i] = [1] * (3 + off) if i == 1 else wrong
        with pytest.raises(ValueError):
            nnv.nnv_conv_forward_grouped(*args, None, stream=0)
        with pytest.raises(ValueError):
            nnv.nnv_cold_stack(*args, None, stream_exec=0)


def test_arguments_of_other_types_are_refused(calls):
    d, other = desc(), (TypeError, ctypes.ArgumentError)
    with pytest.raises(other):
        nnv.nnv_conv_forward(object(), 1, A, A, None, A, None, stream=0)
    with pytest.raises(other):
        nnv.nnv_conv_forward(nnv.Timing(), 1, A, A, None, A, None, stream=0)
    with pytest.raises(other):
        nnv.nnv_conv_forward(d, "direct", A, A, None, A, None, stream=0)
    with pytest.raises(other):
        nnv.nnv_conv_forward_grouped([d, 1], [1, 1], [A, A], [A, A], None, [A, A], None, stream=0)
    with pytest.raises(AttributeError):
        nnv.nnv_conv_forward(d, 1, "x", A, None, A, None, stream=0)
    with pytest.raises(AttributeError):
        nnv.nnv_transform_weights_grouped([d], [1], [None], [A], stream=0)
    with pytest.raises(AttributeError):
        nnv.nnv_conv_forward(d, 3, A, A, None, A, A, stream=0)      # an address has no size


def test_module_argument_counts():
    native = binding._calls()
    with pytest.raises(TypeError):
        native.conv_forward(desc(), 1)
    with pytest.raises(TypeError):
        native.setup(1)
    with pytest.raises(TypeError):
        native.setup(1, 2, 3, 4, 5)


def test_without_a_compiled_module_the_calls_go_through_ctypes(monkeypatch, tmp_path):
    """No module, and none to be built (no headers or no compiler): the library still loads and takes calls."""
    def no_module(*_):
        raise RuntimeError("no headers")
    monkeypatch.setattr(binding, "MODULE_PATH", str(tmp_path / "none.so"))
    monkeypatch.setattr(build, "build_module", no_module)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    with pytest.warns(UserWarning, match="through ctypes"):
        nnv.load()
    assert binding._native is binding._CtypesCalls
    assert status(nnv.nnv_conv_forward, desc(), 1, None, A, None, A, None) == NULL


def test_module_name_carries_the_interpreter():
    assert build.MODULE.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


@pytest.mark.gpu
def test_both_routes_give_the_same_bytes(monkeypatch):
    """Every call of the module on device tensors and the current stream, once compiled and once through ctypes."""
    native, dev = binding._calls(), torch.device("cuda:0")
    assert native is not binding._CtypesCalls
    d = desc()
    gen = torch.Generator(device=dev).manual_seed(31)
    w = torch.randn(16 * 16 * 9, device=dev, generator=gen)
    x = torch.rand(16 * 32 * 32, device=dev, generator=gen)
    bias = torch.randn(16, device=dev, generator=gen)
    kinds = [nnv.DIRECT, nnv.IM2COL_GEMM, nnv.WINO_F2, nnv.WINO_F4]
    n = len(kinds)
    sizes = [nnv.nnv_transformed_bytes(d, k) for k in kinds]

    def outputs():
        txs = [torch.zeros(s, dtype=torch.uint8, device=dev) for s in sizes]
        ys = [torch.zeros(16 * 32 * 32, device=dev) for _ in range(5 * n)]
        need = max([nnv.nnv_workspace_bytes(d, k) for k in kinds] + [nnv.nnv_conv_forward_grouped_workspace_bytes([d] * n, kinds)])
        ws = torch.empty(need, dtype=torch.uint8, device=dev)
        nnv.nnv_transform_weights_grouped([d] * n, kinds, [w] * n, txs)
        one = torch.zeros_like(txs[2])
        nnv.nnv_transform_weights(d, kinds[2], w, one)
        for i, k in enumerate(kinds):
            nnv.nnv_conv_forward(d, k, x, txs[i], bias, ys[i], ws)
            nnv.nnv_conv_forward_relu(d, k, x, txs[i], None, ys[n + i], ws)
            nnv.nnv_conv_forward_static(d, k, x, txs[i], bias, ys[2 * n + i])
        nnv.nnv_conv_forward_grouped([d] * n, kinds, [x] * n, txs, [bias] * n, ys[3 * n:4 * n], ws, flags=nnv.FORWARD_RELU)
        nnv.nnv_cold_stack([d] * n, kinds, [w] * n, [t.clone() for t in txs], [x] * n, ys[4 * n:], ws)
        torch.cuda.synchronize()
        return [t.cpu() for t in txs + [one] + ys]

    compiled = outputs()
    monkeypatch.setattr(binding, "_native", binding._CtypesCalls)
    for a, b in zip(compiled, outputs()):
        assert a.any() and torch.equal(a, b)
