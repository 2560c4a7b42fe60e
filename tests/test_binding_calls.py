"""The extension module of the per-step calls hands the library exactly what the caller passed: its function
addresses are pointed at Python callbacks of the C signatures, no GPU involved."""
import ctypes
import os
import sys
import sysconfig
import types

import pytest

from paper_2504_03661_amd import binding as B
from paper_2504_03661_amd import build as lib_build

vp, i32 = ctypes.c_void_p, ctypes.c_int32
DECODE = ctypes.CFUNCTYPE(i32, *([vp] * 10), ctypes.c_float, vp, vp)
APPEND = ctypes.CFUNCTYPE(i32, vp, vp, vp, i32, *([vp] * 6))


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Stream:
    def __init__(self, raw):
        self.cuda_stream = raw


def recorder(monkeypatch, name, kind, status):
    seen = []
    fn = kind(lambda *a: seen.append(a) or status)
    B.load_library()
    monkeypatch.setattr(B, name, ctypes.cast(fn, vp).value)
    return seen, fn


HIGH = 0xFFFF_8000_0000_1000      # an address with the top bit set


@pytest.mark.parametrize("ctx", [vp(HIGH), HIGH, None])
@pytest.mark.parametrize("stream,raw", [(0, None), (7, 7), (Stream(HIGH), HIGH), (Stream(0), None)])
def test_arguments_arrive_as_passed(monkeypatch, ctx, stream, raw):
    seen, _fn = recorder(monkeypatch, "_decode_at", DECODE, 0)
    B.pq_attn_decode(ctx, Tensor(1), Tensor(HIGH), 3, 4, None, Tensor(0), Tensor(7), None, 9, 1 / 8, Tensor(11), stream)
    at = ctx.value if isinstance(ctx, vp) else ctx
    assert seen == [(at, 1, HIGH, 3, 4, None, None, 7, None, 9, 0.125, 11, raw)]
    for n_new in (0, 1, -1, 2**31 - 1):
        seen, _fn = recorder(monkeypatch, "_append_at", APPEND, 0)
        B.pq_encode_append(ctx, Tensor(1), 2, n_new, None, Tensor(HIGH), Tensor(6), 7, Tensor(8), stream)
        assert seen == [(at, 1, 2, n_new, None, HIGH, 6, 7, 8, raw)]


def test_the_default_stream_is_the_current_one_at_each_call(monkeypatch):
    seen, _fn = recorder(monkeypatch, "_append_at", APPEND, 0)
    for current in (5, 6):
        monkeypatch.setattr(B, "_current_stream", lambda: current)
        B.pq_encode_append(None, 1, 2, 1, None, None, 3, 4, 5)
    assert [a[-1] for a in seen] == [5, 6]


def test_a_status_raises_and_a_wrong_type_is_refused(monkeypatch):
    _seen, _fn = recorder(monkeypatch, "_decode_at", DECODE, -1)
    with pytest.raises(B.PQAttnError):
        B.pq_attn_decode(None, 1, 2, 3, 4, None, None, None, None, None, 1.0, 5, 0)
    seen, _fn = recorder(monkeypatch, "_decode_at", DECODE, 0)
    with pytest.raises(AttributeError):
        B.pq_attn_decode(None, 1.5, 2, 3, 4, None, None, None, None, None, 1.0, 5, 0)
    with pytest.raises(TypeError):
        B.pq_attn_decode(None, 1, 2, 3, 4, None, None, None, None, None, None, 5, 0)
    assert not seen


@pytest.mark.parametrize("missing", [None, "_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_the_current_stream_without_torchs_private_getters(monkeypatch, missing):
    """torch's own accessors are a shortcut: where a torch has none, its public call answers at each call."""
    import torch
    current = [5]
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(current[0]))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 1, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 10 * device + current[0], raising=False)
    for name in ("_raw_stream", "_raw_device"):
        monkeypatch.setattr(B, name, None)
    if missing:
        monkeypatch.delattr(torch._C, missing)
    seen = [B._current_stream()]                        # the first call starts torch's GPU context through the public one
    current[0] = 6
    seen += [B._current_stream(), B._current_stream()]
    assert seen == ([5, 16, 16] if missing is None else [5, 6, 6])


def test_contexts_are_taken_as_ctypes_takes_them(monkeypatch):
    """A pointer object is an address; an object that is none is refused, whatever attributes it has."""
    cell = ctypes.c_int32(5)
    seen = []
    lib = types.SimpleNamespace(pq_attn_decode=DECODE(lambda *a: seen.append(a[0]) or 0),
                                pq_encode_append=APPEND(lambda *a: seen.append(a[0]) or 0))
    B.load_library()
    monkeypatch.setattr(B, "_lib", lib)
    for name in ("_decode_at", "_append_at"):           # (the extension module must not see these)
        monkeypatch.setattr(B, name, 0)
    decode = lambda ctx: B.pq_attn_decode(ctx, 1, 2, 3, 4, None, None, None, None, None, 1.0, 5, 0)
    append = lambda ctx: B.pq_encode_append(ctx, 1, 2, 1, None, None, 3, 4, 5, 0)
    for call in (decode, append):
        call(ctypes.pointer(cell))
        with pytest.raises(ctypes.ArgumentError):
            call(ctypes.c_uint64(64))
    assert seen == [ctypes.addressof(cell)] * 2


def test_the_library_serves_without_the_extension_module(monkeypatch):
    for name in ("_lib", "_calls"):
        monkeypatch.setattr(B, name, None)
    monkeypatch.setitem(sys.modules, B.__package__ + "._pq_calls", None)       # its import raises ModuleNotFoundError
    assert B.load_library() is B._lib and B._calls is None
    assert B.pq_status_string(0)
    seen = []
    monkeypatch.setattr(B, "_lib", types.SimpleNamespace(pq_attn_decode=DECODE(lambda *a: seen.append(a) or 0),
                                                         pq_encode_append=APPEND(lambda *a: seen.append(a) or 0)))
    B.pq_attn_decode(HIGH, Tensor(1), Tensor(HIGH), 3, 4, None, Tensor(0), Tensor(7), None, 9, 1 / 8, Tensor(11), Stream(6))
    B.pq_encode_append(HIGH, Tensor(1), 2, 5, None, Tensor(HIGH), Tensor(6), 7, Tensor(8), 0)
    assert seen == [(HIGH, 1, HIGH, 3, 4, None, None, 7, None, 9, 0.125, 11, 6), (HIGH, 1, 2, 5, None, HIGH, 6, 7, 8, None)]


@pytest.mark.parametrize("missing", ["headers", "compiler"])
def test_the_library_builds_where_the_extension_module_cannot(monkeypatch, tmp_path, missing):
    """hipcc stands in as a command that succeeds; what is looked at is that nothing else is asked for."""
    monkeypatch.setenv("HIPCC", "/bin/true")
    monkeypatch.setattr(lib_build, "CALLS", str(tmp_path / "_pq_calls.so"))
    if missing == "headers":
        monkeypatch.setattr(sysconfig, "get_paths", lambda *a, **k: {"include": str(tmp_path)})
    else:
        monkeypatch.setenv("CXX", str(tmp_path / "no_such_compiler"))
    assert lib_build.build(force=True) == lib_build.LIB
    assert not os.path.exists(lib_build.CALLS)
    assert lib_build.stale() == any(os.path.getmtime(f) > os.path.getmtime(lib_build.LIB) for f in
                                    [os.path.join(lib_build.CSRC, s) for s in lib_build.SOURCES] + lib_build.HEADERS)


def test_the_extension_module_is_named_for_its_interpreter():
    assert os.path.basename(lib_build.CALLS) == "_pq_calls" + sysconfig.get_config_var("EXT_SUFFIX")
