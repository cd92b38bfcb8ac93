"""Failures of the HIP runtime, over the stand-in GPU of tests/host_double: the
runtime keeps the error of a failed call until the thread asks for its last
one, as every kernel launch does, so an error that was reported or that the
library gets by without must be gone by the next launch."""
import ctypes

import numpy as np
import pytest

import host_util as H


def _domain(L, N, nx, ny):
    p, keep = H.params(N, nx, ny, 32)
    d = ctypes.c_void_p()
    rc = L.nplbm_create(ctypes.addressof(p), L.double_stream(), None, 0, ctypes.byref(d))
    return rc, d


@pytest.mark.parametrize("nth", [1, 3])
def test_a_large_readback_without_pinned_memory_leaves_no_error(nth):
    L = H.lib()
    rc, d = _domain(L, 2, 2048, 1900)       # c of 62 MB, moved in chunks
    H.check(rc)
    c = H.even(2, 2048 * 1900)
    H.check(L.nplbm_set_fields(d, H.ptr(c), None))
    H.check(L.nplbm_step(d, 3))
    L.double_fail(b"hipHostMalloc", nth)
    for steps in (3, 4):
        H.check(L.nplbm_get_c(d, H.ptr(c)))
        assert np.all(c == steps)
        H.check(L.nplbm_step(d, 1))
    L.double_fail(b"hipHostFree", 1)
    L.nplbm_destroy(d)
    rc, d = _domain(L, 2, 40, 30)
    H.check(rc)
    c = H.even(2, 1200)
    H.check(L.nplbm_set_fields(d, H.ptr(c), None))
    L.nplbm_destroy(d)


@pytest.mark.parametrize("call", ["hipMemcpyAsync", "hipStreamBeginCapture", "hipGraphLaunch",
                                  "hipMalloc"])
def test_a_reported_error_is_reported_once(call):
    L = H.lib()
    rc, d = _domain(L, 3, 40, 30)
    H.check(rc)
    c = H.even(3, 1200)
    H.check(L.nplbm_set_fields(d, H.ptr(c), None))
    L.double_fail(call.encode(), 1)
    if call == "hipMalloc":
        rc, other = _domain(L, 3, 40, 30)
        assert rc == -3 and not other
    elif call == "hipMemcpyAsync":
        assert L.nplbm_set_fields(d, H.ptr(c), None) == -4
    else:
        assert L.nplbm_step(d, 2) == -4
    H.check(L.nplbm_step(d, 2))
    H.check(L.nplbm_get_c(d, H.ptr(c)))
    assert np.all(c == 2)
    L.nplbm_destroy(d)


def test_admissions_that_fail_do_not_fail_the_next_ones():
    s = H.Server(quantum=4)
    ts = [s.submit(N, 64, 40, 6) for N in (2, 3, 4)]
    s.L.double_fail(b"hipMalloc", 1)
    while s.pump() != (0, 0):
        pass
    assert [s.result(t) for t in ts] == [-3, 6, 6]
    s.close()
