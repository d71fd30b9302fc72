"""How the library would dispatch a launch (zl_launch_route of zl_internal.h), for tests that are about one
kernel or rule: they assert that their sizes reach it."""
import ctypes

from paper_2608_01150_amd import api

HALVES, ONE_LAUNCH, DQ_FIRST, TWO_PER_CU = 1, 2, 4, 8

_fn = api._lib.zl_launch_route
_fn.restype = ctypes.c_int32
_fn.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int, ctypes.c_int32] + [ctypes.c_void_p] * 3


def route(d, heads, head_dim, op, dtype=api.ZL_BF16, q=1 << 40, dout=2 << 40, dq=3 << 40):
    """d: a descriptor's plain data (tests._descs).  q, dout, dq: addresses, never read."""
    desc = api.SegDesc.of(d)
    r = _fn(ctypes.cast(desc.ptr(), ctypes.c_void_p), heads, head_dim, dtype, op, q, dout, dq)
    assert r >= 0, api.last_error()
    return r
