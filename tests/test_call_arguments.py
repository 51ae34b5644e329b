"""The extension that calls the library (csrc/apt_call.c): every kind of argument arrives as the address or integer it stands for, and
what is taken and refused is what ctypes takes and refuses."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig
import threading
import time

import numpy as np
import pytest
import torch

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import build

_apt_call = pytest.importorskip("paper_2504_07494_amd._apt_call", reason="built without a host compiler or Python headers")
ab._step("apt_plan")                                      # (sets the extension up)

SEEN = []


def _function(n, types=None):
    """A C function of n 64-bit arguments that records them and returns the first, cut to an int; its address; the function with the
    given argument types."""
    def record(*args):
        SEEN.append(args)
        return C.c_int(args[0] & 0xffffffff).value
    f = C.CFUNCTYPE(C.c_int, *[C.c_uint64] * n)(record)
    address = C.cast(f, C.c_void_p).value
    typed = C.CFUNCTYPE(C.c_int, *(types or [C.c_uint64] * n))(address)
    typed.keep = f
    return f, address, typed


def _never(*args):
    raise AssertionError("left to ctypes")


@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 7, 8, 12, 13, 17])
def test_as_many_arguments_as_the_calls_have(n):
    f, address, _ = _function(n)
    SEEN.clear()
    assert _apt_call.call(address, b"a" * n, _never, *range(100, 100 + n)) == 100
    assert SEEN == [tuple(range(100, 100 + n))]


def test_arguments_of_a_decode_step_are_converted_here():
    f, address, _ = _function(10)
    tensor, array, view = torch.arange(8), np.arange(8), np.arange(8)[::-2]
    array.setflags(write=False)
    shape = ab.apt_shape()
    SEEN.clear()
    _apt_call.call(address, b"aaaaaisipp", _never, None, 2 ** 63 + 5, tensor[2:], array, view, -1, shape, 7, 9, None)
    assert SEEN == [(0, 2 ** 63 + 5, tensor[2:].data_ptr(), array.__array_interface__["data"][0], view.__array_interface__["data"][0],
                     2 ** 64 - 1, C.addressof(shape), 7, 9, 0)]


class _Stream:                                            # as torch's streams
    _as_parameter_ = C.c_void_p(7)


class _Index:
    def __index__(self):
        return 5


class _Large(C.Structure):
    _fields_ = [("shape", ab.apt_shape), ("more", C.c_int32)]


SHAPE, TENSOR, LARGE, DATES = ab.apt_shape(), torch.arange(4), _Large(), np.array(["2020-01-01"], dtype="datetime64[D]")
NUMBER = C.c_int(3)


@pytest.mark.parametrize("kind,ctype,value,want", [
    # numpy integers, as lengths' own maxima and sizes come, and everything with an index
    (b"i", C.c_int, np.int64(3), 3), (b"i", C.c_int, np.int32(3), 3), (b"i", C.c_size_t, np.uint64(3), 3), (b"i", C.c_int, np.array(3), 3),
    (b"i", C.c_int, torch.tensor(3), 3), (b"i", C.c_int, _Index(), 5), (b"i", C.c_int, True, 1),
    # ctypes integers of the argument's own type
    (b"i", C.c_int, C.c_int(3), 3), (b"i", C.c_size_t, C.c_size_t(3), 3), (b"i", C.c_size_t, C.c_int(3), None),
    (b"i", C.c_int, None, None), (b"i", C.c_int, 1.0, None), (b"i", C.c_int, np.float32(1), None), (b"i", C.c_int, np.arange(2), None),
    (b"i", C.c_int, torch.zeros(2), None), (b"i", C.c_int, "3", None), (b"i", C.c_int, C.c_void_p(3), None),
    # streams: an integer, a ctypes pointer, a stream object
    (b"p", C.c_void_p, 7, 7), (b"p", C.c_void_p, None, 0), (b"p", C.c_void_p, C.c_void_p(7), 7), (b"p", C.c_void_p, _Stream(), 7),
    (b"p", C.c_void_p, np.int64(7), None), (b"p", C.c_void_p, 1.0, None), (b"p", C.c_void_p, torch.zeros(1), None),
    # buffers
    (b"a", C.c_void_p, TENSOR, TENSOR.data_ptr()), (b"a", C.c_void_p, DATES, DATES.ctypes.data), (b"a", C.c_void_p, C.c_void_p(77), 77),
    (b"a", C.c_void_p, C.c_void_p(), 0), (b"a", C.c_void_p, NUMBER, C.addressof(NUMBER)), (b"a", C.c_void_p, SHAPE, C.addressof(SHAPE)),
    (b"a", C.c_void_p, object(), None), (b"a", C.c_void_p, "text", None), (b"a", C.c_void_p, bytes(64), None), (b"a", C.c_void_p, np.int64(7), None),
    # structures: nothing but ctypes objects
    (b"s", C.c_void_p, SHAPE, C.addressof(SHAPE)), (b"s", C.c_void_p, LARGE, C.addressof(LARGE)), (b"s", C.c_void_p, NUMBER, C.addressof(NUMBER)),
    (b"s", C.c_void_p, None, None), (b"s", C.c_void_p, bytes(48), None), (b"s", C.c_void_p, b"short", None),
    (b"s", C.c_void_p, bytearray(48), None), (b"s", C.c_void_p, np.zeros(2, dtype=np.uint8), None), (b"s", C.c_void_p, torch.zeros(48), None)])
def test_taken_and_refused_as_by_ctypes(kind, ctype, value, want):
    f, address, typed = _function(1, [ctype])
    for function in (lambda x: ab._by_ctypes(typed, kind, x),
                     lambda x: _apt_call.call(address, kind, lambda *a: ab._by_ctypes(typed, kind, *a), x)):
        SEEN.clear()
        if want is None:
            with pytest.raises((TypeError, C.ArgumentError)):
                function(value)
            assert not SEEN
        else:
            function(value)
            assert SEEN == [(want,)]


def test_arguments_of_the_calls_themselves():
    """Through the library's own functions, all refused before anything runs on a device: a status is an argument's way there and back."""
    shape = ab.make_shape(128, 1, 128, 16, "f16", 8, 1.0)
    null = [None] * 9
    for stream in (0, None, C.c_void_p(0), _Stream()):
        for B in (1, np.int32(1), np.int64(1), C.c_int(1)):
            with pytest.raises(ab.AptError) as e:
                ab.apt_cache_append(shape, B, *null, stream)
            assert e.value.status == ab.APT_EINVAL
            with pytest.raises(ab.AptError) as e:
                ab.apt_cache_write(shape, B, None, np.int64(4), *null, stream)
            assert e.value.status == ab.APT_EINVAL
        for n in (64, np.int64(64), C.c_size_t(64)):
            with pytest.raises(ab.AptError) as e:
                ab.apt_hybrid_decode_attn(shape, *[None] * 14, n, stream)
            assert e.value.status == ab.APT_EINVAL
        with pytest.raises(ab.AptError) as e:
            ab.apt_plan_upload(None, None, stream)
        assert e.value.status == ab.APT_EINVAL
    for shape in (bytes(48), np.zeros(48, dtype=np.uint8), b"", None):
        with pytest.raises((TypeError, C.ArgumentError)):
            ab.apt_cache_append(shape, 1, *null)
        with pytest.raises((TypeError, C.ArgumentError)):
            ab.apt_plan(shape, np.ones(1, dtype=np.int32), np.zeros(1, dtype=np.uint8), np.zeros(512, dtype=np.int32))


@pytest.mark.parametrize("kinds,args", [(b"aa", (1,)), (b"a", (1, 2)), (b"a" * 18, tuple(range(18)))])
def test_another_number_of_arguments_is_refused(kinds, args):
    f, address, _ = _function(1)
    SEEN.clear()
    with pytest.raises(TypeError):
        _apt_call.call(address, kinds, _never, *args)
    assert not SEEN


def test_an_error_inside_data_ptr_is_not_taken_for_another_kind():
    class Tensor:
        def data_ptr(self):
            raise RuntimeError("no storage")

    f, address, _ = _function(1)
    with pytest.raises(RuntimeError, match="no storage"):
        _apt_call.call(address, b"a", _never, Tensor())


def test_other_threads_run_during_a_call():
    """The called function blocks without touching Python: another thread only gets on if the call has released the interpreter."""
    ticks, stop = [0], threading.Event()

    def tick():
        while not stop.is_set():
            ticks[0] += 1
            time.sleep(0.001)

    other = threading.Thread(target=tick)
    other.start()
    usleep = C.cast(C.CDLL(None).usleep, C.c_void_p).value
    before = ticks[0]
    assert _apt_call.call(usleep, b"i", _never, 500000) == 0
    after = ticks[0]
    stop.set()
    other.join()
    assert after - before >= 5                            # held: at most the tick that the call's own end lets through


def test_without_the_extension_the_calls_go_through_ctypes():
    """In a process of its own, where the extension cannot be imported: the planner, the pool and the library's checks answer the same."""
    script = """
import sys
if "without" in sys.argv:
    sys.modules["paper_2504_07494_amd._apt_call"] = None
import numpy as np
from paper_2504_07494_amd import binding as ab
shape = ab.make_shape(5120, 40, 128, 16, "f16", 64, 0.1)
lens, kinds = np.array([700, 33, 512, 1000], dtype=np.int32), np.array([1, 0, 1, 0], dtype=np.uint8)
blob = np.zeros(ab.apt_plan_max_bytes(shape, 4, 1024) // 4, dtype=np.int32)
info = ab.apt_plan(shape, lens, kinds, blob)
assert ab.apt_pool_free_blocks(ab.apt_pool_create(8, 16, 4, 2)) == 8
try:
    ab.apt_cache_append(shape, np.int64(4), *[None] * 9, 0)
except ab.AptError as e:
    assert e.status == ab.APT_EINVAL
print(info.n_items, info.plan_bytes, hash(blob.tobytes()), ab._step("apt_plan").func is ab._by_ctypes)
"""
    env = dict(os.environ, PYTHONHASHSEED="0", PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    got = [subprocess.run([sys.executable, "-c", script, *words], env=env, text=True, capture_output=True, check=True).stdout.split()
           for words in ([], ["without"])]
    assert got[0][:3] == got[1][:3] and [g[3] for g in got] == ["False", "True"]


def test_the_extension_is_left_out_of_a_build_that_cannot_make_it(monkeypatch, tmp_path):
    monkeypatch.delenv("CC", raising=False)
    assert build.CALL.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    with monkeypatch.context() as m:
        m.setattr(build.shutil, "which", lambda name: f"/usr/bin/{name}")
        m.setenv("CC", "ccache gcc -pipe")
        command = build.extension_command()
        assert command[:3] == ["ccache", "gcc", "-pipe"] and command[-1] == build.CALL
    with monkeypatch.context() as m:
        m.setenv("CC", str(tmp_path / "no such compiler").replace(" ", "_"))
        assert build.extension_command() is None
    with monkeypatch.context() as m:
        m.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
        assert build.extension_command() is None
    with monkeypatch.context() as m:
        m.setattr(build.platform, "machine", lambda: "aarch64")
        assert build.extension_command() is None
