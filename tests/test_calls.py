"""The native argument marshalling (csrc/calls.cpp) against what the binding's functions say they pass: every entry point is replaced by a
recorder, called through the binding, and the recorded C arguments are compared.  No GPU."""
import ctypes

import pytest
import torch

from paper_2509_09090_amd import binding as B

VP, I32, I64, U32, SZ, F32, F64 = (ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint32, ctypes.c_size_t, ctypes.c_float,
                                   ctypes.c_double)


class Sub(torch.Tensor):
    """A subclass is asked through Python."""


def _half(*shape, kind=torch.Tensor):
    t = torch.zeros(shape, dtype=torch.float16)
    return t if kind is torch.Tensor else t.as_subclass(kind)


@pytest.fixture
def recorded(monkeypatch):
    """name -> arguments of the calls made; `status` is what they return."""
    B.lib()
    from paper_2509_09090_amd import _calls
    calls, keep, result = [], [], {"status": 0}

    def address(name):
        types = getattr(B.lib(), name).argtypes

        def record(*args):
            calls.append((name, args))
            return result["status"]
        keep.append(ctypes.CFUNCTYPE(I32, *types)(record))
        return ctypes.cast(keep[-1], VP).value

    monkeypatch.setattr(B, "_native", _calls.Calls(address, lambda: 0x77, B._check))
    yield calls, result
    del keep[:]


@pytest.mark.parametrize("kind", [torch.Tensor, Sub])
def test_arguments_reach_the_library(recorded, kind):
    calls, _ = recorded
    x, wide = _half(6, 64, kind=kind), _half(6, 200, kind=kind)[:, :64]
    rows, u8, i32 = torch.zeros(4, dtype=torch.int32), torch.zeros(6, 32, dtype=torch.uint8), torch.zeros(2, 5, dtype=torch.int32)
    f32, f64, k4 = torch.zeros(2, 16), torch.zeros(2, 26, dtype=torch.float64), _half(2, 20, 4, 8, kind=kind)
    ws, s1 = torch.zeros(24, dtype=torch.float32), _half(6)
    p = lambda t: t.data_ptr()                       # noqa: E731
    handle = ctypes.c_void_p(0x1234560)

    def expect(name, *args):
        got_name, got = calls.pop()
        assert not calls and got_name == name
        assert tuple(got) == args

    B.sqap_attn_scores_batch(s1, k4, 3, 16, f32, ws)
    expect("sqap_attn_scores_batch", p(s1), p(k4), 2, 20, 4, 8, 3, 16, p(f32), p(ws), 96, 0x77)
    B.sqap_prune_topk(f32, 9, i32, stream=5)
    expect("sqap_prune_topk", p(f32), 2, 16, 9, p(i32), 5)
    B.sqap_kept_rows(i32, 30, 4, 16, rows)
    expect("sqap_kept_rows", p(i32), 2, 5, 30, 4, 16, p(rows), 0x77)
    B.sqap_prune_rows(f32, 9, 30, 4, i32, rows)
    expect("sqap_prune_rows", p(f32), 2, 16, 9, 30, 4, p(i32), p(rows), 0x77)
    B.sqap_prune_select(f32, 4, 4, 3, 9, f64, 2, i32)
    expect("sqap_prune_select", p(f32), 2, 4, 4, 3, 9, p(f64), 2, p(i32), 5, None, 0x77)
    B.sqap_quantize_act(wide, rows, u8, s1, flags=1)
    expect("sqap_quantize_act", p(wide), 200, p(rows), 4, 64, 1, p(u8), p(s1), 0x77)
    B.sqap_quantize_act(wide, None, u8, s1)
    expect("sqap_quantize_act", p(wide), 200, None, 6, 64, 0, p(u8), p(s1), 0x77)
    B.sqap_rmsnorm_quantize_act(wide, rows, s1, 0.25, u8, s1, delta=x, flags=1, col_scales=k4, xsum_out=ws, y_out=f32)
    expect("sqap_rmsnorm_quantize_act", p(wide), 200, p(rows), 4, 64, p(x), p(s1), 0.25, 1, p(k4), p(ws), p(f32), p(u8), p(s1), 0x77)
    B.sqap_swiglu_quantize_act(wide, x, u8, s1, h_out=k4)
    expect("sqap_swiglu_quantize_act", p(wide), 200, p(x), 64, 6, 64, None, p(k4), p(u8), p(s1), 0x77)
    B.sqap_rope(wide, rows, 4, 16, 500.5)
    expect("sqap_rope", p(wide), 200, p(rows), 6, 4, 16, 500.5, 0x77)
    B.sqap_rope_append(wide, rows, 4, 16, x)
    expect("sqap_rope_append", p(wide), 200, p(rows), 6, 4, 16, 10000.0, p(x), 64, 0x77)
    B.sqap_attention(wide, x, k4, 4, 16, s1, batch=4)
    expect("sqap_attention", p(wide), 200, p(x), 64, p(k4), 640, 4, 1, 1, 4, 16, p(s1), 1, 0x77)
    B.sqap_decode_attention(s1, rows, 4, 16, wide, 3, x, u8, s1, i32)
    expect("sqap_decode_attention", p(s1), p(rows), 4, 16, 10000.0, p(wide), 200, 3, p(x), p(u8), p(s1), p(i32), 0x77)
    B.sqap_w4a4_linear(u8, s1, B.Weight(None, 1, 1), wide, None, ws)
    expect("sqap_w4a4_linear", p(u8), p(s1), 6, None, p(wide), 200, None, p(ws), 96, 0x77)
    w = B.Weight.__new__(B.Weight)
    w.handle = handle
    B.sqap_w4a4_linear(u8, s1, w, wide, i32, None, stream=9)
    w.handle = None
    expect("sqap_w4a4_linear", p(u8), p(s1), 6, 0x1234560, p(wide), 200, p(i32), None, 0, 9)
    g = B.Group.__new__(B.Group)
    g.handle = handle
    g.run()
    g.handle = None
    expect("sqap_group_run", 0x1234560, 0x77)
    d = B.Decoder.__new__(B.Decoder)
    d.handle = handle
    d.step(s1, rows, 17, x, attn_trace=wide)
    d.handle = None
    expect("sqap_decoder_step", 0x1234560, p(s1), p(rows), 17, p(x), p(wide), 0x77)


def test_refusals(recorded):
    calls, result = recorded
    x, u8, s1, i32 = _half(6, 64), torch.zeros(6, 32, dtype=torch.uint8), _half(6), torch.zeros(2, 5, dtype=torch.int32)
    with pytest.raises(IndexError):
        B.sqap_quantize_act(s1, None, u8, s1)                      # no second dimension
    with pytest.raises(ValueError):
        B.sqap_prune_topk(s1, 2, i32)                              # two dimensions wanted
    with pytest.raises(ValueError):
        B.sqap_swiglu_quantize_act(_half(2, 3, 8), x, u8, s1)
    with pytest.raises(TypeError):
        B.sqap_rope(x, i32, 4.0, 16)
    with pytest.raises(TypeError):
        B.sqap_rope(x, i32, None, 16)
    with pytest.raises(AttributeError):
        B.sqap_rope(x, 3, 4, 16)                                   # no tensor
    with pytest.raises(ZeroDivisionError):
        B.sqap_attention(x, x, x, 4, 16, x, batch=0)
    with pytest.raises(RuntimeError):
        B.sqap_rope(x.to_sparse(), i32, 4, 16)                     # no storage: torch's own error
    with pytest.raises(TypeError):
        B._native.quantize_act(x)
    from paper_2509_09090_amd import _calls
    with pytest.raises(TypeError):
        _calls.Calls()
    assert not calls
    result["status"] = B.EINVAL
    with pytest.raises(B.SqapError) as e:
        B.sqap_quantize_act(x, None, u8, s1)
    assert e.value.status == B.EINVAL


def test_current_stream_is_asked_for_until_one_device_is_known(recorded, monkeypatch):
    calls, _ = recorded
    x, u8, s1 = _half(6, 64), torch.zeros(6, 32, dtype=torch.uint8), _half(6)
    assert B._native.one_device is False
    monkeypatch.setattr(B, "_stream", lambda stream: 0x55)
    monkeypatch.setattr(B.torch.cuda, "device_count", lambda: 1)
    monkeypatch.setattr(B.torch.cuda, "is_initialized", lambda: False)
    assert B._current_stream() == 0x55 and B._native.one_device is False
    monkeypatch.setattr(B.torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(B.torch.cuda, "device_count", lambda: 2)
    assert B._current_stream() == 0x55 and B._native.one_device is False
    B.sqap_quantize_act(x, None, u8, s1)
    assert calls.pop()[1][-1] == 0x77
    monkeypatch.setattr(B.torch.cuda, "device_count", lambda: 1)
    assert B._current_stream() == 0x55 and B._native.one_device is True
    B._forked()
    assert B._native.one_device is False


def test_a_call_that_outlasts_the_interpreter():
    """A daemon thread still in a call when the program ends: the program ends as ever, without an abort."""
    import os
    import subprocess
    import sys
    program = """
import ctypes, sys, threading, time
from paper_2509_09090_amd import binding as B
B.lib()
from paper_2509_09090_amd import _calls
libc = ctypes.CDLL(None)
sleep = ctypes.cast(libc.usleep, ctypes.c_void_p).value
calls = _calls.Calls(lambda name: sleep, lambda: 0, B._check)          # (the handle is how long)
threading.Thread(target=calls.group_run, args=(ctypes.c_void_p(900000), 0), daemon=True).start()
time.sleep(0.2)
class Late:
    def __del__(self):
        libc.usleep(1500000)                                           # without the interpreter's lock, while it ends
sys.modules["late"] = Late()
print("done", flush=True)
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", program], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "done\n", (r.returncode, r.stderr)


@pytest.mark.gpu
def test_native_calls_follow_the_current_stream():
    x, u8, s1 = (_half(6, 64).cuda(), torch.zeros(6, 32, dtype=torch.uint8, device="cuda"), _half(6).cuda())
    seen = []
    for _ in range(2):                                             # the first call may be the one that asks
        B.sqap_quantize_act(x, None, u8, s1)
    from paper_2509_09090_amd import _calls
    keep = []

    def address(name):
        types = getattr(B.lib(), name).argtypes
        keep.append(ctypes.CFUNCTYPE(I32, *types)(lambda *a: seen.append(a[-1]) or 0))
        return ctypes.cast(keep[-1], VP).value
    native = _calls.Calls(address, lambda: B._current_stream(), B._check)
    native.one_device = torch.cuda.device_count() == 1
    side = torch.cuda.Stream()
    native.quantize_act(x, None, u8, s1, 0, None)
    with torch.cuda.stream(side):
        native.quantize_act(x, None, u8, s1, 0, None)
    native.quantize_act(x, None, u8, s1, 0, None)
    assert [v or 0 for v in seen] == [torch.cuda.current_stream().cuda_stream, side.cuda_stream, torch.cuda.current_stream().cuda_stream]
