"""The library's host sources built with g++ over the stand-in GPU of
tests/host_double, for CPU tests of the host logic: scheduling, failures of
the runtime, host copies.  Calls go through the C ABI, as the binding's do.
"""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

import paper_1904_12553_amd as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_LIB = None


def lib():
    global _LIB
    if _LIB is None:
        csrc = os.path.join(ROOT, "paper_1904_12553_amd", "csrc")
        dbl = os.path.join(ROOT, "tests", "host_double")
        with tempfile.TemporaryDirectory() as tmp:
            out = os.path.join(tmp, "libhost.so")
            subprocess.run(
                ["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-pthread", "-Wl,-Bsymbolic",
                 "-I", dbl, "-I", os.path.join(ROOT, "include"), "-I", csrc, "-o", out,
                 os.path.join(dbl, "double.cpp")] +
                [os.path.join(csrc, f) for f in ("nplbm_host.cpp", "nplbm_api.cpp",
                                                 "nplbm_server.cpp", "host_copy.cpp")],
                check=True)
            _LIB = ctypes.CDLL(out)
        vp, sz, i64 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int64
        for name, args, res in (
                ("nplbm_last_error", [], ctypes.c_char_p), ("nplbm_footprint", [vp], sz),
                ("nplbm_create", [vp, vp, vp, sz, vp], ctypes.c_int),
                ("nplbm_set_fields", [vp, vp, vp], ctypes.c_int),
                ("nplbm_step", [vp, i64], ctypes.c_int), ("nplbm_get_c", [vp, vp], ctypes.c_int),
                ("nplbm_get_state", [vp, vp, vp], ctypes.c_int),
                ("nplbm_destroy", [vp], None), ("nplbm_state_bytes", [vp], sz),
                ("nplbm_server_create", [sz, ctypes.c_int32, ctypes.c_int32, vp, vp],
                 ctypes.c_int),
                ("nplbm_submit", [vp, vp, vp, vp, i64, vp], ctypes.c_int),
                ("nplbm_server_pump", [vp, vp], ctypes.c_int),
                ("nplbm_poll", [vp, ctypes.c_uint64, vp], ctypes.c_int),
                ("nplbm_result", [vp, ctypes.c_uint64, vp, vp, vp, vp, vp], ctypes.c_int),
                ("nplbm_server_destroy", [vp], None),
                ("double_fail", [ctypes.c_char_p, ctypes.c_int], None),
                ("double_calls", [ctypes.c_char_p], i64), ("double_reset", [], None),
                ("double_stream", [], vp), ("double_threads", [], ctypes.c_int),
                ("double_unsafe", [], i64), ("double_pinned", [], i64),
                ("double_launches", [], ctypes.c_int), ("double_node_array", [vp], ctypes.c_int),
                ("double_launch", [ctypes.c_int, vp], None)):
            f = getattr(_LIB, name)
            f.argtypes, f.restype = args, res
    _LIB.double_reset()
    return _LIB


def params(N, nx, ny, precision=32, **kw):
    sigma = np.full((N, N), 1e-3)
    return P.nplbm.make_params(N=N, nx=nx, ny=ny, sigma=sigma, rho=np.ones(N),
                               mu=np.full(N, 0.1), precision=precision, **kw)


def even(N, nodes):
    return np.full((N, nodes), 1.0 / N)


def ptr(a):
    return a.ctypes.data


def check(rc):
    assert rc == 0, (rc, _LIB.nplbm_last_error())


def launches():
    """(N, precision, tile rows, domains, from a graph, stream) of each step launch."""
    out = np.empty((_LIB.double_launches(), 6), np.int64)
    for i in range(len(out)):
        _LIB.double_launch(i, ptr(out[i]))
    return [tuple(int(v) for v in row) for row in out]


class Server:
    def __init__(self, budget=1 << 40, slots=8, quantum=4):
        self.L = lib()
        h = ctypes.c_void_p()
        check(self.L.nplbm_server_create(budget, slots, quantum, self.L.double_stream(),
                                         ctypes.byref(h)))
        self.h, self.shape = h, {}

    def submit(self, N, nx, ny, steps, precision=32, **kw):
        p, keep = params(N, nx, ny, precision, **kw)
        c = even(N, nx * ny)
        t = ctypes.c_uint64()
        check(self.L.nplbm_submit(self.h, ctypes.addressof(p), ptr(c), None, steps,
                                  ctypes.byref(t)))
        self.shape[t.value] = (N, nx * ny)
        return t.value

    def pump(self):
        active = ctypes.c_int32()
        return self.L.nplbm_server_pump(self.h, ctypes.byref(active)), active.value

    def poll(self, t):
        s = ctypes.c_int32()
        check(self.L.nplbm_poll(self.h, t, ctypes.byref(s)))
        return s.value

    def result(self, t):
        """The number of steps that the result of a finished request holds, or
        the error code."""
        c = np.empty(self.shape[t])
        rc = self.L.nplbm_result(self.h, t, ptr(c), None, None, None, None)
        if rc:
            return rc
        assert np.all(c == c[0, 0])
        return int(c[0, 0])

    def close(self):
        self.L.nplbm_server_destroy(self.h)
