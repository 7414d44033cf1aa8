"""Argument checks of the internal launchers, made on the host before any
device call (no GPU needed)."""
import ctypes
import os

import pytest

from paper_2311_18715_amd import odmd as B

INVALID_VALUE = 1                 # hipErrorInvalidValue


class PassArgs(ctypes.Structure):                     # pass.h
    _fields_ = [("Us", ctypes.c_void_p), ("x", ctypes.c_void_p), ("y", ctypes.c_void_p), ("partials", ctypes.c_void_p),
                ("st", ctypes.c_void_p), ("n", ctypes.c_int64), ("units", ctypes.c_int64), ("nblk", ctypes.c_int),
                ("ct", ctypes.c_int), ("eout", ctypes.c_void_p), ("threads", ctypes.c_int), ("rows2", ctypes.c_int)]


@pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libodmd.so not built")
@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="the checks are made without a GPU")
def test_a_residual_output_is_not_dropped():
    """The pass by itself has no residual output: asked for one, it must not
    run and leave it unwritten.  The launch that has one needs it, and equal
    partitions of its two sweeps."""
    lib = B.lib()
    one = lib._ZN4odmd11launch_passERKNS_8PassArgsEiiP12ihipStream_tP11ihipEvent_tS6_
    two = lib._ZN4odmd16launch_pass_pairERKNS_8PassArgsES2_iiP12ihipStream_tP11ihipEvent_tS6_
    ints = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    one.argtypes, one.restype = [ctypes.POINTER(PassArgs), *ints], ctypes.c_int
    two.argtypes, two.restype = [ctypes.POINTER(PassArgs), ctypes.POINTER(PassArgs), *ints], ctypes.c_int
    p = PassArgs(n=1000, nblk=2, ct=24, threads=256, eout=1)
    t = PassArgs(n=1000, nblk=2, ct=24, threads=256)
    assert one(p, 0, 24, None, None, None) == INVALID_VALUE
    assert two(t, t, 0, 24, None, None, None) == INVALID_VALUE
    for field in ("n", "nblk", "threads", "rows2"):
        u = PassArgs.from_buffer_copy(t)
        setattr(u, field, getattr(u, field) + 1)
        assert two(p, u, 0, 24, None, None, None) == INVALID_VALUE
