"""The device calls as Python reaches them (csrc/calls.cpp): the same statuses as through ctypes for
arguments that the library refuses before any GPU work, and errors for what is no integer."""
import ctypes
import importlib.machinery
import os
import sys

import pytest
import torch

from paper_1705_01626_amd import build as zvc_build
from paper_1705_01626_amd import zvc

IN, OUT, BYTES, WS = 1 << 20, 2 << 20, 3 << 20, 4 << 20
BIG = 1 << 40

REFUSED = [
    ("zvc_compress", (IN, 100, 3, OUT, BIG, BYTES, WS, BIG, 0)),
    ("zvc_compress", (IN, 100, 4, OUT, 10, BYTES, WS, BIG, 0)),
    ("zvc_compress", (IN + 1, 100, 2, OUT, BIG, BYTES, WS, BIG, 0)),
    ("zvc_compress", (0, 100, 4, OUT, BIG, BYTES, WS, BIG, 0)),
    ("zvc_compress_static", (IN, 1 << 40, 4, OUT, BIG, BYTES, 0)),
    ("zvc_relu_compress", (IN, 100, 4, OUT, BIG, BYTES, WS + 8, BIG, 0)),
    ("zvc_compress_bounded", (IN, 100, 4, 2, OUT, BIG, BYTES, WS, BIG, 0)),
    ("zvc_compressed_size", (IN, 100, 4, BYTES + 4, WS, BIG, 0)),
    ("zvc_decompress", (IN, 1, 100, 4, OUT, WS, BIG, 0)),
    ("zvc_window_compress", (IN, 100, 4, 4097, OUT, BIG, BYTES, BYTES + 64, WS, BIG, 0)),
    ("zvc_window_decompress", (IN, 100, BYTES, 100, 4, 4096, 5, 1, OUT, 0)),
    ("zvc_offload", (IN, 100, 4, OUT, BIG, 0, 10, BYTES, WS, BIG, 0, 0)),
    ("zvc_relu_offload", (IN, 100, 5, OUT, BIG, 0, 10, BYTES, WS, BIG, 0, 0)),
    ("zvc_prefetch", (IN, 3, 100, 4, OUT, BIG, BYTES, WS, BIG, 0, 0)),
    ("zvc_window_count", (100000, 4, 4096)),
    ("zvc_window_elements", (2, 65536)),
]


@pytest.mark.parametrize("name,args", REFUSED)
def test_same_result_as_ctypes(name, args):
    want = getattr(zvc.load(), name)(*args)
    assert getattr(zvc._native(), name)(*args) == want
    if name not in ("zvc_window_count", "zvc_window_elements"):
        assert want != zvc.ZVC_OK


def test_what_is_no_call_is_an_error():
    calls = zvc._native()
    with pytest.raises(TypeError):
        calls.zvc_window_count(100000, 4)
    with pytest.raises(TypeError):
        calls.zvc_window_count(100000, 4, "4096")
    with pytest.raises(TypeError):
        calls.zvc_window_count(1.5, 4, 4096)
    assert calls.zvc_window_count(-1, 4, 4096) == zvc.load().zvc_window_count(-1, 4, 4096)
    with pytest.raises(ImportError):
        calls.open("/nowhere/libzvc.so")
    assert calls.zvc_window_elements(4, 4096) == 1024


@pytest.mark.parametrize("size", [1000.0, "1000", None, (1000,)])
def test_what_is_no_integer_raises_the_error_of_ctypes(size):
    """... which callers of the functions may catch."""
    with pytest.raises(ctypes.ArgumentError):
        zvc.load().zvc_window_count(size, 4, 4096)
    with pytest.raises(ctypes.ArgumentError):
        zvc.zvc_window_count(size, 4)
    buffer = torch.zeros(8192, dtype=torch.uint8)
    with pytest.raises(ctypes.ArgumentError):
        zvc._native().zvc_decompress(buffer.data_ptr(), size, 100, 4, buffer.data_ptr(), buffer.data_ptr(), 0, 0)


def test_a_call_while_another_thread_loads(monkeypatch):
    """The library is loaded and its entry is not yet: a call in between makes it ready itself."""
    zvc.load()
    monkeypatch.setattr(zvc, "_calls", None)
    assert zvc.zvc_window_count(100000, 4) == 98


def test_without_the_extension_module_calls_go_through_ctypes(monkeypatch):
    """The library needs the HIP compiler alone; a machine that built no more than that makes every call."""
    monkeypatch.setattr(zvc, "_calls", None)
    monkeypatch.setitem(sys.modules, "paper_1705_01626_amd._calls", None)
    monkeypatch.setattr(zvc, "_lib", None)
    assert zvc.load().zvc_mask_bytes(65) == 12
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert zvc.zvc_window_count(100000, 4) == 98
    for name, args in REFUSED[:3]:
        assert getattr(zvc._native(), name)(*args) == getattr(zvc.load(), name)(*args) != zvc.ZVC_OK


def test_the_module_is_built_for_this_interpreter_only(tmp_path, monkeypatch):
    calls = importlib.import_module("paper_1705_01626_amd._calls")
    assert calls.__file__ == zvc_build.CALLS and calls.__file__.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])
    assert "python" in os.path.basename(calls.__file__) or "cp3" in os.path.basename(calls.__file__)
    # no headers of the interpreter: nothing is built, and that is no error
    monkeypatch.setattr(zvc_build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert zvc_build.build_calls(str(tmp_path / "out.so")) is None and not os.listdir(tmp_path)


def test_a_newer_header_is_built_again(tmp_path):
    """The signatures of include/zvc.h are compiled into both files."""
    old, new = tmp_path / "a.so", tmp_path / "zvc.h"
    old.write_text(""), new.write_text("")
    os.utime(old, (1000, 1000)), os.utime(new, (2000, 2000))
    assert zvc_build._older(str(old), str(new)) and not zvc_build._older(str(new), str(old))
    assert zvc_build._older(str(tmp_path / "not there.so"), str(new))
