"""The binding's native caller of the chain entry points (CPU only): every
argument reaches the C function as ctypes passed it, and what is no handle,
buffer set or number is refused."""
import ctypes

import numpy as np
import pytest

from paper_2608_12123_amd import rc_cohort as rc

SIG = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32,
                       ctypes.c_int, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_void_p)


@pytest.fixture(scope="module")
def call():
    rc.load_library()
    return rc._call


@pytest.mark.parametrize("handle,seen_handle", [
    (None, None), (ctypes.c_void_p(None), None), (ctypes.c_void_p(0x7FFF12345678), 0x7FFF12345678), (0x1234, 0x1234)])
@pytest.mark.parametrize("stream", [None, 0, 2, 0x7FFFFFFFF000])
@pytest.mark.parametrize("step0", [0, 5, 0xFFFFFFFE, 1 << 32, -1, np.uint32(7)])
def test_arguments_arrive(call, handle, seen_handle, stream, step0):
    seen = []
    buffers = rc.RcBuffers(1, 2, 3, 4, 5, 6, 77)

    @SIG
    def fn(*a):
        got = ctypes.cast(a[1], ctypes.POINTER(rc.RcBuffers)).contents
        seen.append(a[:1] + tuple(getattr(got, f) for f, _ in rc.RcBuffers._fields_) + a[2:])
        return 3

    addr = ctypes.cast(fn, ctypes.c_void_p).value
    assert call(addr, handle, buffers, step0, 16, 1, 2, 9, stream) == 3
    assert seen == [(seen_handle, 1, 2, 3, 4, 5, 6, 77, int(step0) & 0xFFFFFFFF, 16, 1, 2, 9, stream or None)]


def test_refused(call):
    @SIG
    def fn(*a):
        raise AssertionError("called")

    addr = ctypes.cast(fn, ctypes.c_void_p).value
    b = rc.RcBuffers()
    for args in [(addr, "h", b, 0, 1, 0, 0, 1, 0), (addr, None, None, 0, 1, 0, 0, 1, 0),
                 (addr, None, (ctypes.c_char * 4)(), 0, 1, 0, 0, 1, 0), (addr, None, b, 0.5, 1, 0, 0, 1, 0),
                 (addr, None, b, 0, "1", 0, 0, 1, 0), (addr, None, b, 0, 1, 0, 0, 1)]:
        with pytest.raises(TypeError):
            call(*args)
    assert rc.rc_cohort_run_chain(None, b, 0, 1, 0, 0, 1, stream=0, check=False) == rc.RC_E_INVALID
    with pytest.raises(rc.RcError):
        rc.rc_cohort_run_chain_noalloc(None, b, 0, 1, 0, 0, 1, stream=0)


# Forms of an argument: whatever ctypes takes is taken with the same value,
# whatever it refuses is refused with its error.
FORMS = [
    ("n_steps", ctypes.c_uint32(8)), ("n_steps", np.int64(8)), ("n_steps", True), ("n_steps", 8.0),
    ("n_steps", "8"), ("n_steps", None), ("mode", ctypes.c_int(1)), ("mode", ctypes.c_uint32(1)),
    ("step0", 1 << 35), ("step0", 2.0), ("cohort_end", ctypes.c_uint32(3)),
    ("h", ctypes.c_uint64(0x1234)), ("h", np.array([0x1234], dtype=np.uint64)), ("h", bytearray(8)),
    ("h", -1), ("h", 1 << 70), ("buffers", bytearray(56)), ("buffers", np.zeros(7, dtype=np.uint64)),
    ("buffers", (ctypes.c_char * 56)()), ("buffers", None),
]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("name,value", FORMS, ids=lambda v: v if isinstance(v, str) else type(v).__name__)
def test_forms_are_those_of_ctypes(call, monkeypatch, name, value, noalloc):
    seen = []

    @SIG
    def fn(*a):
        seen.append(a)
        return 0

    class Lib:  # the entry points as load_library declares them
        pass
    real = rc.load_library()
    addr = ctypes.cast(fn, ctypes.c_void_p).value
    proto = ctypes.CFUNCTYPE(ctypes.c_int)
    for n in ("rc_cohort_run_chain", "rc_cohort_run_chain_noalloc"):
        f = proto(addr)
        f.argtypes, f.restype = getattr(real, n).argtypes, ctypes.c_int
        setattr(Lib, n, staticmethod(f))
    monkeypatch.setattr(rc, "_lib", Lib)
    monkeypatch.setattr(rc, "_fn_run_chain", addr)
    monkeypatch.setattr(rc, "_fn_run_chain_noalloc", addr)
    buffers = rc.RcBuffers(1, 2, 3, 4, 5, 6, 77)
    args = {"h": ctypes.c_void_p(0x4321), "buffers": buffers, "step0": 5, "n_steps": 16, "mode": 1,
            "cohort_begin": 2, "cohort_end": 9, "stream": 0}
    args[name] = value
    run = rc.rc_cohort_run_chain_noalloc if noalloc else rc.rc_cohort_run_chain

    def outcome(native):
        monkeypatch.setattr(rc, "_call", call if native else None)
        seen.clear()
        try:
            run(**args)
        except Exception as e:
            assert not seen
            return type(e)
        return list(seen)
    assert outcome(True) == outcome(False)
