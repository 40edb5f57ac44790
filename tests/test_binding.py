"""The native call forms of the binding against its general path: what is not of the plain form is left to the general path,
which accepts or refuses it; what is of the plain form gives the same tensors."""
import enum
import sys
import time
import warnings

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2605_20315_amd as mq
from paper_2605_20315_amd import _lib, ops


class _General:
    """Takes the native module's place: every call goes to the general path."""

    def __getattr__(self, name):
        return lambda *args: None


class _Recorder:
    """The native module, noting which of its forms were called and whether each took its call (returned no None)."""

    def __init__(self):
        self.module, self.calls = _lib.load_binding(), []

    def __getattr__(self, name):
        form = getattr(self.module, name)

        def call(*args):
            result = form(*args)
            self.calls.append((name, result is not None))
            return result
        return call


def test_a_declined_call_costs_little():
    """Against the 6 to 17 us that the general path takes: 0.1 us declined by a return value, 3.7 by a C++ exception."""
    fast = _lib.load_binding()
    x, u8, f = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(4, 32, dtype=torch.uint8), torch.zeros(1)
    for call in (lambda: fast.quantize(x, f, None, None, 0), lambda: fast.bf16_gemm_ws(x, x, None, 0, None),
                 lambda: fast.linear(x, f, u8, u8, f, 0, None, None, None, 0, None)):
        best = float("inf")
        for _ in range(20):
            start = time.perf_counter()
            for _ in range(1000):
                call()
            best = min(best, (time.perf_counter() - start) * 1e3)
        assert best < 1.5, f"{best:.2f} us"


def test_calls_that_are_not_of_the_plain_form_are_left_alone():
    fast = _lib.load_binding()
    x, u8, f = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(4, 32, dtype=torch.uint8), torch.zeros(1)
    assert fast.global_scale(x, None) is None                      # not on the GPU
    assert fast.quantize(x, f, None, None, 0) is None
    assert fast.quantize(None, f, None, None, 0) is None           # not a tensor
    assert fast.quantize_silu_mul(x, f, None, None, 0) is None
    assert fast.quantize_rmsnorm(x, x, 1e-6, f, None, None, 0) is None
    assert fast.relayout(u8, u8, 0, 1) is None
    assert fast.gemm_ws(u8, u8, f, u8, u8, f, None, 0, None, 0) is None
    assert fast.linear(x, f, u8, u8, f, 0, None, None, None, 0, None) is None
    assert fast.bf16_gemm_ws(x, x, None, 0, None) is None
    with pytest.raises(TypeError):
        fast.bf16_gemm_ws(x, x)
    with pytest.raises(mq.MixQuantError, match="GPU"):
        mq.nvfp4_linear(x, f, u8, u8, f)


def _x(M, K, seed=0, ld=None):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(M, ld or K, device="cuda", generator=g).to(torch.bfloat16)[:, :K]


def _flat(r):
    return [t for p in r for t in _flat(p)] if isinstance(r, (tuple, list)) else [r]


def _calls(M, N, K, ld, out):
    """(the native forms that a call goes through, the outputs given to it, the call)"""
    x, w = _x(M, K, 1, ld), _x(N, K, 2)
    ax, aw = mq.nvfp4_global_scale(x), mq.nvfp4_global_scale(w)
    w0, ws = w[0].clone(), torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    dtype = torch.float32 if out == mq.MQ_OUT_FP32 else torch.bfloat16
    for layout in (mq.MQ_LAYOUT_LINEAR, mq.MQ_LAYOUT_KTILE):
        wc, wsc = mq.nvfp4_quantize(w, aw, layout=layout)
        xc, xsc = mq.nvfp4_quantize(x, ax, layout=layout)
        for given in (False, True):
            y = torch.empty(M, N + 8, dtype=dtype, device="cuda")[:, :N] if given else None
            c = torch.empty(M, K // 2, dtype=torch.uint8, device="cuda") if given else None
            s = torch.empty(M, K // 16, dtype=torch.uint8, device="cuda") if given else None
            yield ["quantize"], [c, s], lambda: mq.nvfp4_quantize(x, ax, c, s, layout)
            yield ["quantize_rmsnorm"], [c, s], lambda: mq.nvfp4_quantize_rmsnorm(x, w0, 1e-6, ax, c, s, layout)
            yield ["linear"], [y, c, s, ws], lambda: (mq.nvfp4_linear(x, ax, wc, wsc, aw, out, y, c, s, layout, ws if given else None), c, s)
            yield ["gemm_ws"], [y, ws], lambda: mq.nvfp4_gemm_ws(xc, xsc, ax, wc, wsc, aw, ws, out, y, layout)
            yield ["bf16_gemm_ws"], [y, ws], lambda: mq.bf16_gemm_ws(x, w, ws if given else None, out, y)
        yield ["quantize_silu_mul"], [], lambda: mq.nvfp4_quantize_silu_mul(w, aw, layout=layout)
        yield ["relayout"], [], lambda: mq.nvfp4_relayout(wc, wsc, layout, 1 - layout)
    yield ["global_scale"], [], lambda: mq.nvfp4_global_scale(x)
    a = torch.empty(1, device="cuda")
    yield ["global_scale"], [a], lambda: mq.nvfp4_global_scale(w, a)


def _spoil(given, sizes):
    """No right bytes are left in the given outputs, nor in the blocks that the allocator may hand out next."""
    for t in given:
        if t is not None:
            t.fill_(0xA5 if t.dtype == torch.uint8 else float("nan"))
    held = [torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda") for n in sizes for _ in range(4)]
    del held


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,ld", [(1, 16, 128, None), (1, 64, 256, 512), (33, 72, 256, 264), (64, 512, 1024, None)])
@pytest.mark.parametrize("out", [mq.MQ_OUT_BF16, mq.MQ_OUT_FP32])
def test_native_and_general_path_give_the_same_tensors(monkeypatch, M, N, K, ld, out):
    sizes = [4] + [r * K // d for r in (M, N) for d in (2, 4, 16, 32)] + [M * N * 2, M * N * 4]
    for i, (forms, given, call) in enumerate(_calls(M, N, K, ld, out)):
        results = []
        for path in (_General(), _Recorder()):
            _spoil(given, sizes)
            with monkeypatch.context() as m:
                m.setattr(ops, "_fast", path)
                made = [t for t in _flat(call()) if t is not None]
            results.append((made, [t.clone() for t in made]))  # both stay alive: no block is handed out twice
        assert path.calls == [(f, True) for f in forms], i     # (by the native form, and by nothing else)
        (_, want), (_, got) = results
        assert len(got) == len(want), i
        for g, w in zip(got, want):
            assert g.dtype == w.dtype and g.shape == w.shape and torch.equal(g, w), i


@pytest.mark.gpu
def test_given_outputs_come_back_and_refusals_stay(monkeypatch):
    x, w = _x(8, 128), _x(16, 128)
    y = torch.empty(8, 16, dtype=torch.bfloat16, device="cuda")
    assert mq.bf16_gemm_ws(x, w, None, mq.MQ_OUT_BF16, y) is y
    a = torch.empty(1, device="cuda")
    assert mq.nvfp4_global_scale(x, a) is a
    for general in (False, True):
        if general:
            monkeypatch.setattr(ops, "_fast", _General())
        with pytest.raises(mq.MixQuantError, match="nvfp4_quantize: MQ_ERR_ARG"):
            mq.nvfp4_quantize(x, a, layout=7)
        with pytest.raises(mq.MixQuantError, match="bf16_gemm_ws: MQ_ERR_ALIGN"):
            mq.bf16_gemm_ws(x, w, None, mq.MQ_OUT_BF16, torch.empty(8, 20, dtype=torch.bfloat16, device="cuda")[:, 4:])
        with pytest.raises(AssertionError):
            mq.bf16_gemm_ws(x.float(), w, None)
        with pytest.raises(mq.MixQuantError, match="contiguous"):
            mq.bf16_gemm_ws(x.t(), w, None)


@pytest.mark.gpu
def test_current_stream_is_used(monkeypatch):
    native = _Recorder()
    monkeypatch.setattr(ops, "_fast", native)
    x, w = _x(64, 1024), _x(256, 1024)
    want = mq.bf16_gemm_ws(x, w, None)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    y = torch.zeros_like(want)
    graph = torch.cuda.CUDAGraph()
    mq.mq_init()
    with torch.cuda.graph(graph, stream=side):   # a launch on any other stream would not be captured
        mq.bf16_gemm_ws(x, w, None, mq.MQ_OUT_BF16, y)
    assert native.calls == [("bf16_gemm_ws", True)] * 2 and not y.any()
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


class _Refused(Exception):
    pass


class _NoAllocation(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is torch.ops.aten.empty.memory_format:
            raise _Refused("no allocation here")
        return func(*args, **(kwargs or {}))


@pytest.mark.gpu
def test_an_error_raised_by_a_dispatch_mode_reaches_the_caller():
    x, w = _x(8, 128), _x(16, 128)
    a = mq.nvfp4_global_scale(x)
    c, s = mq.nvfp4_quantize(x, a)
    for call in (lambda: mq.nvfp4_global_scale(x), lambda: mq.nvfp4_quantize(x, a), lambda: mq.bf16_gemm_ws(x, w, None),
                 lambda: mq.nvfp4_linear(x, a, c, s, a), lambda: mq.nvfp4_relayout(c, s, 0, 1)):
        with _NoAllocation(), pytest.raises(_Refused, match="no allocation here"):
            call()
    y = torch.empty(8, 16, dtype=torch.bfloat16, device="cuda")
    with _NoAllocation():  # nothing to allocate
        assert mq.bf16_gemm_ws(x, w, None, mq.MQ_OUT_BF16, y) is y


class _Layout(enum.IntEnum):
    LINEAR = mq.MQ_LAYOUT_LINEAR
    KTILE = mq.MQ_LAYOUT_KTILE


@pytest.mark.gpu
def test_forms_that_the_general_path_accepts_are_taken(monkeypatch):
    """An output vector for one row, a whole number as eps, members of an IntEnum: the same results as the general path."""
    x, w = _x(1, 128), _x(16, 128)
    a, w0, y = mq.nvfp4_global_scale(x), w[0].clone(), torch.empty(16, dtype=torch.bfloat16, device="cuda")
    calls = {"bf16_gemm_ws": lambda: mq.bf16_gemm_ws(x, w, None, mq.MQ_OUT_BF16, y.zero_()),
             "quantize_rmsnorm": lambda: mq.nvfp4_quantize_rmsnorm(x, w0, 1, a, layout=_Layout.KTILE),
             "quantize": lambda: mq.nvfp4_quantize(x, a, layout=_Layout.KTILE)}
    for name, call in calls.items():
        with monkeypatch.context() as m:
            m.setattr(ops, "_fast", _General())
            want = [t.clone() for t in _flat(call())]
        with monkeypatch.context() as m:
            native = _Recorder()
            m.setattr(ops, "_fast", native)
            got = _flat(call())
            assert native.calls == [(name, True)]
        assert len(got) == len(want) and all(torch.equal(g, v) for g, v in zip(got, want)), name


def test_cpu_tensors_are_refused_with_no_library_loaded(monkeypatch):
    x, f = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(1)
    monkeypatch.setattr(ops, "_fast", ops._Unbound())
    monkeypatch.setattr(_lib, "load", lambda: pytest.fail("a library was loaded"))
    for call in (lambda: mq.nvfp4_global_scale(x), lambda: mq.nvfp4_quantize(x, f), lambda: mq.bf16_gemm_ws(x, x, None)):
        with pytest.raises(mq.MixQuantError, match="GPU"):
            call()


@pytest.mark.parametrize("content", [None, b"no library"])
def test_a_binding_that_is_missing_or_does_not_load_takes_no_call(monkeypatch, tmp_path, content):
    path = tmp_path / "_binding.so"
    if content:
        path.write_bytes(content)
        monkeypatch.setitem(sys.modules, "paper_2605_20315_amd._binding", None)  # its import raises ImportError
        monkeypatch.delattr(mq, "_binding", raising=False)
    monkeypatch.setattr(_lib, "BINDING_PATH", str(path))
    with warnings.catch_warnings(record=True) as seen:
        warnings.simplefilter("always")
        fast = _lib.load_binding()
    assert len(seen) == (content is not None)
    x = torch.zeros(4, 64, dtype=torch.bfloat16)
    assert fast.global_scale(x, None) is None and fast.bf16_gemm_ws(x, x, None, 0, None) is None


@pytest.mark.gpu
def test_calls_without_the_native_part_of_the_binding(monkeypatch, tmp_path):
    x, w = _x(8, 128), _x(16, 128)
    a = mq.nvfp4_global_scale(x)
    want = _flat([mq.nvfp4_quantize(x, a), mq.bf16_gemm_ws(x, w, None)])
    monkeypatch.setattr(ops, "_fast", ops._Unbound())
    monkeypatch.setattr(_lib, "BINDING_PATH", str(tmp_path / "_binding.so"))
    got = _flat([mq.nvfp4_quantize(x, a), mq.bf16_gemm_ws(x, w, None)])
    assert isinstance(ops._fast, _lib.NoBinding) and all(torch.equal(g, v) for g, v in zip(got, want))
