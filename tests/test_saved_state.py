"""A saved state holds the same bytes whichever kernel stepped the domain and
whatever its memory held: the padding of its rows is zeros."""
import ctypes
import os

import numpy as np
import pytest

import host_util as H
import workloads as W


@pytest.mark.parametrize("N,nx,ny,nz,bits,pad", [(3, 37, 5, 1, 64, 0), (2, 32, 6, 1, 32, 0),
                                                 (4, 33, 4, 4, 32, 0), (2, 32, 6, 1, 32, 7),
                                                 (3, 40, 5, 1, 32, 45)])
def test_padding_of_a_saved_state_is_zero(N, nx, ny, nz, bits, pad, monkeypatch):
    if pad:
        monkeypatch.setenv("NPLBM_ROW_PAD", str(pad))
    L = H.lib()
    p, keep = H.params(N, nx, ny, bits, nz=nz)
    nbytes = L.nplbm_footprint(ctypes.addressof(p))
    mem = np.full(nbytes + 256, 0xA5, np.uint8)          # device memory of the stand-in
    base = -(-H.ptr(mem) // 256) * 256
    d = ctypes.c_void_p()
    H.check(L.nplbm_create(ctypes.addressof(p), None, base, nbytes, ctypes.byref(d)))
    c = H.even(N, nx * ny * nz)
    H.check(L.nplbm_set_fields(d, H.ptr(c), None))
    blob = np.zeros(L.nplbm_state_bytes(d), np.uint8)
    t = ctypes.c_int64()
    H.check(L.nplbm_get_state(d, H.ptr(blob), ctypes.byref(t)))
    L.nplbm_destroy(d)
    size, pitch, rows, M = bits // 8, -(-nx // 32) * 32, ny * nz, N - 1
    planes = (M * (15 if nz > 1 else 9), 14 if nz > 1 else 8, M + (3 if nz > 1 else 2))
    at = 0
    for G, n in enumerate(planes):
        row = (n * pitch + pad) * size
        group = blob[at:at + rows * row].reshape(rows, row)
        assert not np.any(group[:, n * pitch * size:])
        cols = group[:, :n * pitch * size].reshape(rows, n, pitch * size)
        assert not np.any(cols[:, :, nx * size:])
        body = cols[:, :, :nx * size].copy()
        if G == 0:
            body[0, 0, :8] = 0xA5                        # the step count of the stand-in
        assert np.all(body == 0xA5)
        at += rows * row
    assert at == len(blob)


def _state(w, precision, env, steps, **over):
    from tests.gpu_util import gpu_domain
    saved = {k: os.environ.pop(k, None) for k in env}
    os.environ.update(env)
    try:
        d = gpu_domain(w, precision=precision, **over)
    finally:
        for k, v in saved.items():
            os.environ.pop(k, None)
            if v is not None:
                os.environ[k] = v
    d.step(steps)
    out = d.get_state()
    d.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("N,over", [(2, {}), (5, {"grad_scheme": 1}), (8, {"force_form": 1})])
def test_saved_states_of_tiles_and_strips_are_equal(N, over):
    import paper_1904_12553_amd as P
    sig = {"sigma_range": (0.95e-3, 1.05e-3)} if N > 5 else {}
    for nx, ny in ((33, 21), (300, 290)):
        w = W.random_smooth(N, nx, ny, seed=1400 + N + nx, wall_y=True, accept=P.accepts, **sig)
        print(f"case saved state N={N} {nx}x{ny} {over}", flush=True)
        for precision in (64, 32):
            a, ta = _state(w, precision, {"NPLBM_TILE": "8"}, 5, **over)
            b, tb = _state(w, precision, {"NPLBM_TILE": "0"}, 5, **over)
            assert ta == tb == 5 and np.array_equal(a, b), precision


@pytest.mark.gpu
def test_saved_states_of_node_and_marching_kernels_are_equal():
    import paper_1904_12553_amd as P
    w = W.random_smooth3d(3, 37, 20, 9, seed=1450, wall_z=True, accept=P.accepts)
    print("case saved state N=3 37x20x9", flush=True)
    for precision in (64, 32):
        a, _ = _state(w, precision, {"NPLBM_TY3": "0"}, 5)
        b, _ = _state(w, precision, {"NPLBM_TY3": "4"}, 5)
        assert np.array_equal(a, b), precision
