"""The C array of the 3-D node kernels takes the place of the read-back planes:
a domain needs no more memory with them than with the marching kernel, and
read-backs between steps change nothing."""
import ctypes

import numpy as np
import pytest

import workloads as W


@pytest.mark.parametrize("N,nx,ny,nz,bits", [(2, 64, 40, 20, 32), (4, 100, 84, 60, 64),
                                             (5, 65, 150, 150, 64), (5, 5, 9, 6, 64),
                                             (3, 192, 192, 192, 32)])
def test_footprint_does_not_depend_on_the_kernel(N, nx, ny, nz, bits, monkeypatch):
    import paper_1904_12553_amd as P
    kw = dict(N=N, nx=nx, ny=ny, nz=nz, precision=bits, sigma=W.uniform_sigma(N, 1e-3),
              rho=np.ones(N), mu=np.full(N, 0.1))
    sizes = set()
    for ty in (None, "0", "4"):
        monkeypatch.delenv("NPLBM_TY3", raising=False)
        if ty:
            monkeypatch.setenv("NPLBM_TY3", ty)
        sizes.add(P.footprint(**kw))
    assert len(sizes) == 1 and sizes.pop() > 0


def test_the_array_fits_for_every_row_length():
    import host_util as H
    L = H.lib()
    for nx in list(range(4, 70)) + [112, 113, 127, 128, 129, 224, 225, 256, 1000]:
        for N in (2, 3, 4, 5):
            for bits in (32, 64):
                p, keep = H.params(N, nx, 9, bits, nz=5)
                assert L.double_node_array(ctypes.addressof(p)), (nx, N, bits)


@pytest.mark.gpu
@pytest.mark.parametrize("N,nx,ny,nz", [(3, 37, 20, 9), (2, 4, 7, 5), (5, 6, 9, 5), (4, 130, 9, 6)])
def test_read_backs_between_steps_change_nothing(N, nx, ny, nz, monkeypatch):
    import paper_1904_12553_amd as P
    from tests.gpu_util import gpu_domain
    w = W.random_smooth3d(N, nx, ny, nz, seed=1500 + nx, wall_z=True, accept=P.accepts)
    print(f"case read-backs between steps N={N} {nx}x{ny}x{nz}", flush=True)
    for precision in (64, 32):
        monkeypatch.setenv("NPLBM_TY3", "4")
        march = gpu_domain(w, precision=precision)
        march.step(8)
        want = march.macro()
        monkeypatch.setenv("NPLBM_TY3", "0")
        d = gpu_domain(w, precision=precision)
        for steps in (1, 2, 5):
            d.macro()
            d.diagnostics()
            d.laplace(nx / 2, ny / 2, 1.0, 2.0, zc=nz / 2)
            d.step(steps)
        for _ in range(2):
            got = d.macro()
            assert all(np.array_equal(a, b) for a, b in zip(got, want)), precision
        d.set_fields(w.c, w.u)
        d.step(8)
        assert all(np.array_equal(a, b) for a, b in zip(d.macro(), want)), precision
        march.close()
        d.close()
