"""What the native way into the C boundary hands over, and which arguments it leaves to the general way (no GPU): a C function of
this test stands in for the boundary's."""
import ctypes
import threading
import types

import numpy as np
import pytest
import torch

from paper_2605_06472_amd import binding

SEEN = []


@ctypes.CFUNCTYPE(ctypes.c_int, *([ctypes.c_uint64] * 11))
def _record(*args):
    SEEN.append(args)
    return -7


def _call(kinds, *args):
    SEEN.clear()
    fn = binding.fast(types.SimpleNamespace(f=_record), "f", kinds, binding.Shape)
    return fn(*args), (SEEN[0] if SEEN else None)


def test_every_kind_arrives():
    shape = binding.make_shape(3, 8, 2, 128, 16, 100, 7, "bf16")
    t, lens = torch.zeros(4), np.array([5, 6, 7], np.int32)
    stream = types.SimpleNamespace(cuda_stream=99)
    rc, seen = _call("spppiNnt", shape, t, 1 << 63, None, lens, -3, stream)
    assert rc == -7
    assert seen[0] == ctypes.addressof(shape)
    assert seen[1:4] == (t.data_ptr(), 1 << 63, 0)
    assert seen[4] == lens.ctypes.data and seen[5] == 3
    assert ctypes.c_int32(seen[6] & 0xffffffff).value == -3 and seen[7] == 99
    assert _call("t", 77)[1][0] == 77


def test_read_only_lengths_are_plain():
    a = np.arange(5, dtype=np.int32)
    a.setflags(write=False)
    assert _call("i", a)[1][0] == a.ctypes.data


@pytest.mark.parametrize("form", [np.arange(10, dtype=np.int32)[::2], np.arange(5, dtype=np.int64), np.arange(5, dtype=">i4"), np.arange(5, dtype=np.uint32),
                                  np.arange(5, dtype=np.float32), np.arange(4, dtype=np.int32).reshape(2, 2), np.zeros(0, np.int32), [1, 2], torch.arange(5)],
                         ids=["strided", "int64", "big_endian", "uint32", "float32", "2d", "empty", "list", "torch"])
def test_lengths_that_need_converting_are_left_alone(form):
    assert _call("i", form) == (None, None)


@pytest.mark.parametrize("kind,value", [("p", "text"), ("p", 1 << 64), ("p", np.zeros(3)), ("s", 5), ("s", ctypes.c_int(3)), ("n", 2.5), ("n", None), ("t", "text")])
def test_other_forms_are_left_alone(kind, value):
    assert _call(kind, value) == (None, None)


def test_wrong_number_of_arguments_and_kinds():
    with pytest.raises(TypeError):
        _call("pp", 1)
    with pytest.raises(ValueError):
        _call("px", 1, 2)


def test_binding_functions_raise_as_before():
    shape = binding.make_shape(1, 8, 2, 128, 16, 100, 7, "bf16")
    with pytest.raises(binding.PbkvError) as e:            # refused by the boundary, through the native way
        binding.append_kv(shape, None, 16, 16, 16, np.array([1], np.int32), np.array([1], np.int32), stream=0)
    assert e.value.code == -1
    with pytest.raises(binding.PbkvError):                 # the same with lengths that need converting
        binding.append_kv(shape, None, 16, 16, 16, [1], [1], stream=0)
    with pytest.raises(AttributeError):
        binding.append_kv(shape, "text", 16, 16, 16, np.array([1], np.int32), np.array([1], np.int32), stream=0)


def test_threads_call_at_once():
    """The interpreter is not held during the call: two calls wait for each other inside."""
    meet = threading.Barrier(2, timeout=20)
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *([ctypes.c_uint64] * 11))(lambda *a: meet.wait() * 0)
    call = binding.fast(types.SimpleNamespace(f=fn), "f", "n", binding.Shape)
    out = []
    threads = [threading.Thread(target=lambda: out.append(call(1))) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert out == [0, 0]


def test_a_forked_child_leaves_the_stream_to_torch(monkeypatch):
    """torch refuses to name a current device in a forked child of a process that uses the GPU: there the native way asks
    nothing by itself and the general way raises."""
    import os

    from paper_2605_06472_amd import _calls

    def current_device():
        if os.getpid() != parent:
            raise RuntimeError("forked")
        return 3

    parent = os.getpid()
    monkeypatch.setattr(binding, "_torch", None)
    monkeypatch.setattr(torch.cuda, "current_device", current_device)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device, raising=False)
    try:
        assert _call("t", None) == (None, None)                # torch has not been asked yet
        assert binding._stream(None) == 73
        assert _call("t", None)[1][0] == 73
        child = os.fork()
        if child == 0:
            try:
                left = _call("t", None) == (None, None)
                with pytest.raises(RuntimeError):
                    binding._stream(None)
                os._exit(0 if left else 1)
            finally:
                os._exit(2)
        assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 0
        assert _call("t", None)[1][0] == 73
    finally:
        _calls.torch(None, None)


def test_without_the_extension_the_message_says_how_to_build(tmp_path):
    """libpbkv.so alone, or beside the extension of another interpreter: the hint that a missing library gets."""
    import os
    import shutil
    import subprocess
    import sys
    package = tmp_path / "paper_2605_06472_amd"
    package.mkdir()
    for name in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(binding.HERE, name), package / name)
    os.symlink(binding.LIB_PATH, package / "libpbkv.so")
    (package / "_calls.cpython-37m-x86_64-linux-gnu.so").write_bytes(b"another interpreter's")
    r = subprocess.run([sys.executable, "-c", "from paper_2605_06472_amd import binding; binding.load()"], cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode and "ImportError" in r.stderr and "python -m paper_2605_06472_amd.build" in r.stderr, r.stderr


def test_the_extension_is_named_for_its_interpreter():
    import importlib.machinery

    from paper_2605_06472_amd import _calls
    assert _calls.__file__.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])
