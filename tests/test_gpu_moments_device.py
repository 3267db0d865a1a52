"""lbm_moments_device into the caller's arrays: written by the kernel where it
can store there, copied where it cannot (host memory, an address that is no
multiple of 8, arrays that overlap); every way gives lbm_moments' values, and
only the arrays that were asked for are written."""
import ctypes as C
import sys

import numpy as np
import pytest

from lbm_inputs import configs as cfg

from _hip import DeviceArray, hip

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("storage", ["f64", "f32dev", "f16node"])
@pytest.mark.parametrize("where", ["device", "pinned", "odd address", "overlap"])
def test_moments_device(where, storage):
    from paper_1908_09235_amd import lbm as L
    p = cfg.cfg1("mls", "A")
    n = p.nx * p.ny
    say(f"[gpu] moments into {where} arrays, {storage}")
    H = hip()
    with L.Domain(p, storage=storage, history_capacity=64) as d:
        d.step(5)
        want = [w.ravel() for w in d.moments()]
        if where == "pinned":
            host = C.c_void_p()
            H.hipHostMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t, C.c_uint]
            H.hipHostFree.argtypes = [C.c_void_p]
            assert H.hipHostMalloc(C.byref(host), 24 * n, 0) == 0
            try:
                L.lbm_moments_device(d.h, *[host.value + 8 * n * k for k in range(3)])
                L.lbm_sync(d.h)
                got = np.ctypeslib.as_array(C.cast(host, C.POINTER(C.c_double)),
                                            (3, n)).copy()
            finally:
                H.hipHostFree(host)
            assert all(np.array_equal(g, w) for g, w in zip(got, want))
            return
        buf = DeviceArray(np.full(3 * n + 1, -7.0))
        try:
            off = 4 if where == "odd address" else 0
            ptr = [buf.ptr.value + off + 8 * n * k for k in range(3)]
            if where == "overlap":
                ptr[2] = ptr[1]  # the later array wins
            L.lbm_moments_device(d.h, *ptr)
            raw = buf.get().view(np.uint8)
            got = raw[off:off + 24 * n].copy().view(np.float64).reshape(3, n)
            if where == "overlap":
                assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[2])
                return
            assert all(np.array_equal(g, w) for g, w in zip(got, want))
        finally:
            buf.free()
        if where == "device":
            buf = DeviceArray(np.full(3 * n, -7.0))
            try:
                L.lbm_moments_device(d.h, None, buf.ptr.value + 8 * n, None)
                got = buf.get().reshape(3, n)
            finally:
                buf.free()
            assert np.array_equal(got[1], want[1])
            assert (got[0] == -7.0).all() and (got[2] == -7.0).all()
