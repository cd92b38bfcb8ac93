"""The state has one layout.  NPLBM_LAYOUT=soa, which asked for planes one
after the other (a layout that the step kernels do not address), changes
neither the plan of a domain nor its results."""
import ctypes

import numpy as np
import pytest

import host_util as H
import workloads as W


@pytest.mark.parametrize("nz", [1, 12])
def test_the_environment_names_no_other_layout(nz, monkeypatch):
    L = H.lib()
    p, keep = H.params(4, 40, 30, 64, nz=nz)
    sizes = []
    for layout in (None, "soa"):
        if layout:
            monkeypatch.setenv("NPLBM_LAYOUT", layout)
        d = ctypes.c_void_p()
        H.check(L.nplbm_create(ctypes.addressof(p), None, None, 0, ctypes.byref(d)))
        sizes.append((L.nplbm_footprint(ctypes.addressof(p)), L.nplbm_state_bytes(d)))
        L.nplbm_destroy(d)
    assert sizes[0] == sizes[1]


@pytest.mark.gpu
@pytest.mark.parametrize("N,nx,ny,nz", [(2, 5, 9, 1), (3, 100, 41, 1), (3, 20, 9, 6)])
def test_results_do_not_depend_on_it(N, nx, ny, nz, monkeypatch):
    import paper_1904_12553_amd as P
    from tests.gpu_util import gpu_domain
    make = W.random_smooth3d if nz > 1 else W.random_smooth
    w = make(N, nx, ny, *([nz] if nz > 1 else []), seed=1100 + nx, accept=P.accepts)
    print(f"case layout N={N} {nx}x{ny}x{nz}", flush=True)
    for precision in (64, 32):
        out = []
        for layout in (None, "soa"):
            monkeypatch.delenv("NPLBM_LAYOUT", raising=False)
            if layout:
                monkeypatch.setenv("NPLBM_LAYOUT", layout)
            d = gpu_domain(w, precision=precision)
            d.step(11)
            out.append(d.macro())
            d.close()
        assert all(np.array_equal(a, b) for a, b in zip(*out)), precision
