"""The C call path of the per-layer functions hands over what the ctypes path does, for every argument type it takes itself,
and leaves the others to that path."""
import ctypes
import enum
import os
import sysconfig

import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3

torch = pytest.importorskip("torch")
SIG = ("s3_decode_step", "s3_decode_step_static", "s3_kv_append", "s3_decode_attention", "s3_kv_fill_batch")


class Recorder:
    """Functions of the library's signatures that keep their arguments and return a status of their own."""

    def __init__(self):
        self.seen, self.keep, self.handle = {}, [], type("Handle", (), {})()
        for k, name in enumerate(SIG):
            res, args = s3.SIGNATURES[name]
            pointers = (s3._pi32, s3._pi64, ctypes.POINTER(ctypes.c_void_p))
            plain = [ctypes.c_void_p if a in pointers else a for a in args]

            def body(*values, name=name, k=k, args=args):
                # (arrays by what they hold: the two paths have copies of their own)
                held = [list(ctypes.cast(v, a)[:values[2]]) if a in pointers and v else v for v, a in zip(values, args)]
                self.seen.setdefault(name, []).append(held)
                return -10 - k

            fn = ctypes.CFUNCTYPE(res, *plain)(body)
            self.keep.append(fn)
            proto = ctypes.CFUNCTYPE(res, *args)
            setattr(self.handle, name, proto(ctypes.cast(fn, ctypes.c_void_p).value))


@pytest.fixture
def recorder(monkeypatch):
    r = Recorder()
    real = s3._connect()
    monkeypatch.setattr(s3, "_lib", r.handle)
    monkeypatch.setattr(s3, "_call", None)
    s3._connect()
    yield r
    lib = ctypes.CDLL(s3.LIB_PATH)  # the extension is one per process: back to the library
    real.connect(ctypes.c_void_p, *[ctypes.cast(getattr(lib, f), ctypes.c_void_p).value for f in SIG])


def calls(arena, ptrs, dtype, scale, stream):
    a, b, c, d, e, f, g = ptrs
    return {"s3_decode_step": lambda: s3.s3_decode_step(arena, 3, 7, a, b, c, d, e, f, dtype, scale, g, stream),
            "s3_decode_step_static": lambda: s3.s3_decode_step_static(arena, 3, 7, a, b, c, d, e, f, dtype, scale, g, stream),
            "s3_kv_append": lambda: s3.s3_kv_append(arena, 3, 7, a, b, c, d, stream),
            "s3_decode_attention": lambda: s3.s3_decode_attention(arena, 3, 7, a, b, c, d, dtype, scale, stream),
            "s3_kv_fill_batch": lambda: s3.s3_kv_fill_batch(arena, 3, IDS, LENS, [a, b, c], [d, e, f], stream)}


IDS, LENS = np.array([4, 0, 9], np.int32), np.array([17, 0, 250], np.int32)
TENSORS = [torch.zeros(8, dtype=torch.int16) for _ in range(7)]
HIGH = 0xFFFF_8000_1234_5678
CASES = {
    "tensors": (TENSORS, s3.S3_F32, 0.0, 0),
    "no lengths": (TENSORS[:6] + [None], s3.S3_BF16, 0.125, HIGH),
    "addresses": ([16 * i for i in range(1, 6)] + [HIGH, None], s3.S3_F16, 1e-3, 1),
    "numpy arrays": ([np.zeros(4, np.int64) for _ in range(7)], s3.S3_F32, 0.0, 0),
    "whole number as scale": (TENSORS, s3.S3_F32, 1, 0),
    "numpy numbers": (TENSORS, np.int64(s3.S3_BF16), np.float32(0.5), 0),
    "stream none": (TENSORS, s3.S3_F32, 0.0, None),
}


@pytest.mark.parametrize("case", CASES, ids=list(CASES))
def test_the_call_path_passes_what_ctypes_passes(recorder, monkeypatch, case):
    ptrs, dtype, scale, stream = CASES[case]
    arena = ctypes.c_void_p(0x7F00_0000_1000)
    fast = calls(arena, ptrs, dtype, scale, stream)
    for k, name in enumerate(SIG):
        assert fast[name]() == -10 - k

    class Refusing:  # everything goes the ctypes way
        step = step_static = append = attention = fill = staticmethod(lambda *a: None)

    monkeypatch.setattr(s3, "_call", Refusing)
    for k, name in enumerate(SIG):
        assert fast[name]() == -10 - k
        one, two = recorder.seen[name]
        assert one == two, (name, one, two)


@pytest.mark.parametrize("ids,lens,rows", [([4, 0, 9], [1, 2, 3], TENSORS[:3]), (IDS.astype(np.int64), LENS, TENSORS[:3]), (IDS, LENS, tuple(TENSORS[:3])),
                                           (np.repeat(IDS, 2)[::2], LENS, TENSORS[:3]), (IDS, LENS, TENSORS[:2]), (IDS[:0], LENS[:0], [])],
                         ids=["lists", "64 bits", "tuple", "strided", "a row short", "none"])
def test_newcomers_in_other_containers(recorder, ids, lens, rows):
    """What the call path does not take itself reaches the library all the same, as ctypes passes it."""
    arena = ctypes.c_void_p(16)
    assert s3.s3_kv_fill_batch(arena, 0, ids, lens, rows, rows, 0) == -14
    held = recorder.seen["s3_kv_fill_batch"][0]
    n = len(ids)
    want = [t.data_ptr() for t in rows] + [None] * (n - len(rows))
    assert held[2] == n and (n == 0 or (held[3] == list(ids) and held[4] == list(lens) and held[5] == want == held[6]))


def test_what_is_no_pointer_is_refused_as_before(recorder):
    for bad in (calls(ctypes.c_void_p(16), ["x"] + TENSORS[1:], s3.S3_F32, 0.0, 0), calls(ctypes.c_void_p(16), [2.5] + TENSORS[1:], s3.S3_F32, 0.0, 0)):
        for name in SIG:
            with pytest.raises(TypeError):
                bad[name]()
    assert not recorder.seen


class Handle(ctypes.c_void_p):
    pass


NO_ARENA = {"c_int": ctypes.c_int(5), "c_uint64": ctypes.c_uint64(9), "c_size_t": ctypes.c_size_t(16), "enum member": enum.Enum("Colour", {"RED": 5}).RED,
            "any object with a value": type("Boxed", (), {"value": 16})(), "float": 1.5, "tensor": TENSORS[0]}


@pytest.mark.parametrize("what", NO_ARENA, ids=list(NO_ARENA))
def test_what_is_no_arena_is_refused_as_before(recorder, what):
    for name, call in calls(NO_ARENA[what], TENSORS, s3.S3_F32, 0.0, 0).items():
        with pytest.raises(ctypes.ArgumentError):
            call()
    assert not recorder.seen


@pytest.mark.parametrize("arena,address", [(ctypes.c_void_p(), None), (None, None), (16, 16), (Handle(16), 16)], ids=["null", "none", "number", "subclass"])
def test_the_arenas_that_ctypes_takes(recorder, arena, address):
    for name, call in calls(arena, TENSORS, s3.S3_F32, 0.0, 0).items():
        assert call() == -10 - SIG.index(name)
        assert recorder.seen[name][0][0] == address


def test_the_extension_is_named_for_its_interpreter(recorder, monkeypatch, tmp_path):
    """Another interpreter does not load it: it looks for a file of its own, and says how to build one."""
    from paper_2306_06000_amd import build

    assert build.CALL_LIB == s3.CALL_PATH and s3.CALL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert sysconfig.get_config_var("SOABI") in os.path.basename(s3.CALL_PATH)
    monkeypatch.setattr(s3, "_call", None)
    monkeypatch.setattr(s3, "CALL_PATH", str(tmp_path / "_s3call.other.so"))
    with pytest.raises(RuntimeError, match="is missing: build it"):
        s3.s3_kv_append(ctypes.c_void_p(16), 0, 1, *TENSORS[:4])
