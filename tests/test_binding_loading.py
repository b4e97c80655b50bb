"""What the Python binding needs to load and which arguments its step calls take (no GPU: every call returns
before a launch)."""
import ctypes as C
import importlib.util
import os
import shutil
import sys

import pytest

from paper_2505_00347_amd import solo


def fresh_binding(tmp_path, native):
    """A second copy of the binding, in a folder of its own, with the native module or without."""
    solo.lib()
    os.makedirs(tmp_path / "lib")
    shutil.copy(solo.__file__, tmp_path / "solo.py")
    os.symlink(solo.LIB_PATH, tmp_path / "lib" / "libsolo.so")
    if native:
        shutil.copy(solo.NATIVE_PATH, tmp_path / "lib")
    spec = importlib.util.spec_from_file_location("solo_copy", tmp_path / "solo.py")
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


class Number:
    def __init__(self, value):
        self._as_parameter_ = value


@pytest.mark.parametrize("native", (True, False))
def test_the_library_serves_an_interpreter_without_the_native_module(tmp_path, native):
    b = fresh_binding(tmp_path, native)
    assert b.solo_code_words(2560, 3) == 256 and "success" in b.solo_strerror(0)
    cfg = b.make_config(2, 3, 128, 1)
    good = [16, None, 16, None, 16, 16, 16, 16, 16]
    assert b.solo_adamw_step_mp(*good, 0, 1, cfg) == b.SOLO_OK
    assert b.solo_adamw_step_mp(*good, 100, 0, cfg, stream=0, check=False) == b.SOLO_E_INVALID
    assert b.solo_adamw_step(16, 20, *good[4:], 100, 1, cfg, stream=0, check=False) == b.SOLO_E_INVALID
    assert b.solo_adamw_step_multi(16, 1, 0, 0, None, 1, cfg) == b.SOLO_OK
    assert b.solo_adamw_step_multi(8, 1, 1, 0, None, 1, cfg, stream=0, check=False) == b.SOLO_E_INVALID


@pytest.mark.parametrize("native", (True, False))
def test_arguments_that_ctypes_takes(tmp_path, native):
    """Integer objects of ctypes, _as_parameter_, and streams whose handle is one of those or None."""
    b = fresh_binding(tmp_path, native)
    cfg = b.make_config()
    good = [16, None, 16, None, 16, 16, 16, 16, 16]
    assert b.solo_adamw_step_mp(*good, C.c_uint64(0), C.c_uint64(1), cfg) == b.SOLO_OK
    assert b.solo_adamw_step_mp(*good, 0, Number(1), cfg) == b.SOLO_OK
    for stream in (Stream(None), Stream(C.c_void_p(0)), Stream(0), 0):      # (step 0 is refused before a launch)
        assert b.solo_adamw_step_mp(*good, 100, 0, cfg, stream=stream, check=False) == b.SOLO_E_INVALID
        assert b.solo_adamw_step_multi(16, C.c_uint32(1), C.c_uint64(1), 0, None, 0, cfg, stream=stream,
                                       check=False) == b.SOLO_E_INVALID
    with pytest.raises(C.ArgumentError):
        b.solo_adamw_step_mp(*good, 100, 1.5, cfg, stream=0)


def test_a_thread_that_finds_the_library_loaded_finds_all_of_it(tmp_path):
    """At no instruction of the loading is the library set and a step call not."""
    b = fresh_binding(tmp_path, True)
    calls = [name for name in ("_step", "_multi", "_native") if hasattr(b, name)]
    torn = []

    def trace(frame, event, arg):
        if frame.f_code.co_filename != b.__file__:
            return None
        frame.f_trace_opcodes = True
        if b._lib is not None and any(getattr(b, name) is None for name in calls):
            torn.append(frame.f_lineno)
        return trace

    before = sys.gettrace()
    sys.settrace(trace)
    try:
        b.lib()
    finally:
        sys.settrace(before)
    assert calls and b._lib is not None and not torn


def test_a_state_steps_the_buffers_it_names(monkeypatch):
    """SoloState.step() steps what buffers() returns, also of a subclass that returns others."""
    class Elsewhere(solo.SoloState):
        def __init__(self):
            self.n, self.cfg, self.m_codes = 7, solo.make_config(), None

        def buffers(self):
            return 1, 2, 3, 4, 5

    solo.lib()
    calls = []
    monkeypatch.setattr(solo, "_step", lambda *args: calls.append(args) or solo.SOLO_OK)
    state = Elsewhere()
    assert state.step(11, 12, 13, stream=14, param_bf16=15, grad_scale=16) == solo.SOLO_OK
    assert calls == [(11, 15, 12, 16, 1, 2, 3, 4, 5, 7, 13, state.cfg, 14)]
