"""The extension module of the per-step calls marshals as the ctypes binding does: every call with all arguments valid but
an impossible size (no kernel is launched, so no GPU is needed) returns the C library's status; wrong argument
kinds raise and leave nothing behind."""
import pytest
import torch

import paper_2512_00956_amd.binding as P


@pytest.fixture(scope="module")
def F():
    return P._load_fast()


def _t(*shape, dtype=torch.uint8):
    return torch.zeros(shape, dtype=dtype)


X, Y, T, Q, S = _t(4, 40, dtype=torch.bfloat16), _t(4, 64, dtype=torch.bfloat16), _t(64), _t(4, 20), _t(64)
CALLS = [
    ("quantize_act", (X, T, Q, S, None, None, 0)),
    ("linear", (Q, S, Q, S, Y, None, 0, None)),
    ("linear", (Q, S, Q, S, Y, P.default_fmt(layout=1), 0, 40)),
    ("layer_decode", (X, T, Q, S, Y, S, None, 0)),
    ("layer_decode_static", (X, T, Q, S, Y, None, 0)),
    ("quantize_act_nvfp4", (X, T, T, Q, S, 0, None, 0)),
    ("linear_nvfp4", (Q, S, T, Q, S, T, Y, 0, 0, 0, None)),
    ("quantize_act_int4", (X, T, Q, S, 0, None, 0)),
    ("linear_int4", (Q, S, Q, S, Y, 0, 0, 0, None)),
]


@pytest.mark.parametrize("name,args", CALLS)
def test_status_of_an_impossible_size(F, name, args):
    assert getattr(F, name)(*args) == 2                       # K = 40: WUSH_ERR_SHAPE
    null = (None,) + args[1:] if name.startswith("linear") and args[-1] is not None else None
    if null:
        assert getattr(F, name)(*null) == 1                   # WUSH_ERR_NULL


@pytest.mark.parametrize("name,args", CALLS)
def test_calls_without_the_module(monkeypatch, name, args):
    """Where there is no module for the running Python, the same functions through ctypes return the same status."""
    import sys
    monkeypatch.setattr(P, "_fast", None)
    monkeypatch.setitem(sys.modules, "paper_2512_00956_amd._wush_call", None)      # importing it raises ImportError
    monkeypatch.delattr("paper_2512_00956_amd._wush_call", raising=False)
    calls = P._load_fast()
    assert calls.__name__.endswith("_ctypes_call")
    test_status_of_an_impossible_size(calls, name, args)
    with pytest.raises(P.WushError):
        P.wush_linear(Q, S, Q, S, Y, stream=0)


def test_the_build_does_without_a_host_compiler(monkeypatch, tmp_path):
    from paper_2512_00956_amd import build
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CALL_LIB", str(tmp_path / "_wush_call.so"))
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.build_call_module() is None and not list(tmp_path.iterdir())


@pytest.mark.parametrize("name,args", CALLS)
def test_wrong_arguments_raise(F, name, args):
    fn = getattr(F, name)
    with pytest.raises(TypeError):
        fn(*args[:-1])
    with pytest.raises(AttributeError):
        fn(*((object(),) + args[1:]))
    with pytest.raises((TypeError, AttributeError)):
        fn(*(args[:-1] + ("x",)))


def test_format_descriptor_is_checked(F):
    with pytest.raises((TypeError, BufferError)):
        F.linear(Q, S, Q, S, Y, b"short", 0, 40)
    for other in (bytes(P.default_fmt()), torch.zeros(6, dtype=torch.int32).numpy(), 24):
        with pytest.raises(TypeError):
            F.linear(Q, S, Q, S, Y, other, 0, 40)             # the right bytes are not the right type
    bad = P.default_fmt()
    bad.block = 16
    assert F.linear(Q, S, Q, S, Y, bad, 0, 64) == 4           # WUSH_ERR_FMT
    with pytest.raises(ValueError):
        F.quantize_act(_t(4), T, Q, S, None, None, 0)


def test_a_forked_child_asks_torch_for_its_stream(monkeypatch):
    """A stream handle read past torch.cuda.current_stream() would not notice that CUDA cannot be used behind a fork: torch
    refuses there, and so must a call made in the child of a process whose calls have run."""
    import os

    def refuse(*_):
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    monkeypatch.setattr(P, "_raw_stream", lambda: 0x1234)
    assert P._current_stream() == 0x1234
    pid = os.fork()
    if pid == 0:
        code = 1
        try:
            P._current_stream()
        except RuntimeError:
            code = 0
        finally:
            os._exit(code)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert P._current_stream() == 0x1234
