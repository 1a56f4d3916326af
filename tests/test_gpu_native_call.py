"""The native marshalling of the tensor calls against the Python marshalling it
stands in for: the same bits from the same C-ABI call, the same errors, and the
Python path for everything but plain tensors."""
from __future__ import annotations

import pytest

from .gpu_util import require_gpu

pytestmark = pytest.mark.gpu


class _Declines:
    """A native module that declines every call."""

    def __getattr__(self, name):
        return lambda *args: None


def _both(pk, monkeypatch, call):
    """call() natively (which must not decline) and through Python."""
    from paper_1904_05347_amd import binding
    native = binding._native or binding._load_native()
    answers = []

    class Watch:
        def __getattr__(self, name):
            def f(*args):
                r = getattr(native, name)(*args)
                answers.append(r is not None)
                return r
            return f

    monkeypatch.setattr(binding, "_native", Watch())
    first = call()
    used = pk.last_config_name()
    assert answers == [True]
    monkeypatch.setattr(binding, "_native", _Declines())
    second = call()
    assert pk.last_config_name() == used
    monkeypatch.setattr(binding, "_native", native)
    return first, second


def test_native_calls_equal_python_calls(monkeypatch):
    torch, pk = require_gpu()
    g = torch.Generator(device="cuda").manual_seed(1)

    def rand(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    a, b, c0, d = rand(70, 1030)[:, :1027], rand(45, 1027), rand(70, 45), rand(70, 3)
    x, w = rand(2, 13, 11, 20), rand(3, 3, 20, 24)
    ws = torch.empty(1 << 20, device="cuda")
    calls = [
        lambda: pk.gemm(a, b, trans_b=True),
        lambda: pk.gemm(a, b, c0.clone(), alpha=2, beta=0.5, trans_b=True, workspace=ws),
        lambda: pk.gemm(a, d, trans_a=True),
        lambda: pk.conv2d_fwd(x, w),
        lambda: pk.conv2d_fwd(x, w, stride=2, padding="VALID"),
        lambda: pk.conv2d_fwd(x, w, stride=(2, 1), padding=(0, 1, 2, 1), out=torch.empty(2, 7, 11, 24, device="cuda"),
                              workspace=ws),
        lambda: pk.conv2d_winograd(x, w, tile=4),
        lambda: pk.conv2d_winograd(x, w, padding="VALID", workspace=ws),
    ]
    for i, call in enumerate(calls):
        first, second = _both(pk, monkeypatch, call)
        assert first.shape == second.shape and torch.equal(first, second), i


def test_native_calls_decline_and_raise_as_before(monkeypatch):
    torch, pk = require_gpu()
    from paper_1904_05347_amd import binding
    a = torch.ones(8, 8, device="cuda")
    x, w = torch.ones(1, 5, 5, 4, device="cuda"), torch.ones(3, 3, 4, 4, device="cuda")
    bad = [
        lambda: pk.gemm(a.double(), a), lambda: pk.gemm(a.cpu(), a), lambda: pk.gemm(a, a[:4]),
        lambda: pk.gemm(a, a, beta=1.0), lambda: pk.gemm(a, a, beta=1e-50), lambda: pk.gemm(a, a, torch.ones(4, 8, device="cuda")),
        lambda: pk.gemm(a.t()[:, :4], a), lambda: pk.gemm(a, a, a),
        lambda: pk.gemm(a[:1].expand(8, 8), a), lambda: pk.gemm(a, a.as_strided((8, 8), (4, 1)), trans_b=True),
        lambda: pk.gemm(a, a, a[:1].expand(8, 8)), lambda: pk.conv2d_fwd(x[0], w),
        lambda: pk.conv2d_fwd(x, w[:, :, :3]), lambda: pk.conv2d_fwd(x, w, padding="WIDE"),
        lambda: pk.conv2d_fwd(x, w, stride=0), lambda: pk.conv2d_fwd(x, w, out=x),
        lambda: pk.conv2d_winograd(x, w, tile=3), lambda: pk.conv2d_winograd(x, torch.ones(5, 5, 4, 4, device="cuda")),
        lambda: pk.conv2d_winograd(x, w, workspace=torch.empty(4, device="cuda")),
    ]
    native = binding._native or binding._load_native()
    for i, call in enumerate(bad):
        seen = []
        for mod in (native, _Declines()):
            monkeypatch.setattr(binding, "_native", mod)
            with pytest.raises(Exception) as e:
                call()
            seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], i
    monkeypatch.setattr(binding, "_native", native)

    # a tensor subclass and an active mode take the Python path
    class Sub(torch.Tensor):
        pass

    s = a.as_subclass(Sub)
    assert native.gemm(s, a, None, 1.0, 0.0, False, False, None) is None
    assert torch.equal(pk.gemm(s, a).as_subclass(torch.Tensor), pk.gemm(a, a))

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    with Mode():
        assert native.gemm(a, a, None, 1.0, 0.0, False, False, None) is None
        r = pk.gemm(a, a)
    assert torch.equal(r, pk.gemm(a, a))


def test_native_call_runs_on_the_current_stream():
    torch, pk = require_gpu()
    a = torch.ones(512, 512, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        pk.gemm(a, a)
        with torch.cuda.graph(g, stream=s):  # a call on another stream would end the capture
            c = pk.gemm(a, a)
    for _ in range(3):
        c.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert bool((c == 512).all())


def test_native_call_raises_a_failed_launch_once():
    """A launch the runtime refuses is reported, not tried again: with beta, what
    ran before it would run twice."""
    import ctypes

    torch, pk = require_gpu()
    from paper_1904_05347_amd import binding
    native = binding._native or binding._load_native()
    lib = binding.load()
    addresses = [ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in binding._NATIVE_ENTRIES]
    calls = []
    i64, f32, ptr, ch = ctypes.c_int64, ctypes.c_float, ctypes.c_void_p, ctypes.c_char

    @ctypes.CFUNCTYPE(ctypes.c_int, ch, ch, i64, i64, i64, f32, ptr, i64, ptr, i64, f32, ptr, i64, ptr,
                      ctypes.c_size_t, ptr)
    def refuses(*args):
        calls.append(args)
        return binding.PK_ERR_LAUNCH

    a, c = torch.ones(8, 8, device="cuda"), torch.ones(8, 8, device="cuda")
    native.bind(ctypes.cast(refuses, ctypes.c_void_p).value, *addresses[1:], binding._check)
    try:
        with pytest.raises(pk.PkError) as e:
            pk.gemm(a, a, c, beta=1.0)
    finally:
        native.bind(*addresses, binding._check)
    assert e.value.status == binding.PK_ERR_LAUNCH and len(calls) == 1 and bool((c == 1).all())
