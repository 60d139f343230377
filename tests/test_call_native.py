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
