"""The D3Q15 node kernels against the marching kernel and the 3-D oracle:
both evaluate the same expressions per node, so after any number of steps c,
u and p are bitwise equal (NPLBM_TY3 = 0 asks for the node kernels, 4 for
the marching one), and in FP64 they match the oracle within 1e-10 max-abs,
the bound of every FP64 parity test.  Sizes sit where a row of whole cache
lines or a workgroup of 256 nodes can go wrong: rows of a few nodes, one node
past a line, planes below and above a workgroup, walls in z, and both kinds
of stores (states within the 256 MB cache and one beyond it)."""
import os

import numpy as np
import pytest

import workloads as W
from oracle import OracleSim3D
from oracle.accept import oracle_accepts
from tests.gpu_util import gpu_domain, maxabs

pytestmark = pytest.mark.gpu


def _macro(w, precision, steps, ty):
    saved = os.environ.pop("NPLBM_TY3", None)
    os.environ["NPLBM_TY3"] = ty
    try:
        d = gpu_domain(w, precision=precision)
    finally:
        os.environ.pop("NPLBM_TY3", None)
        if saved is not None:
            os.environ["NPLBM_TY3"] = saved
    d.step(steps)
    out = d.macro()
    d.close()
    return out


@pytest.mark.parametrize("N,nx,ny,nz", [(2, 4, 4, 4), (3, 5, 9, 6), (4, 33, 8, 5), (5, 32, 16, 4),
                                        (2, 65, 7, 9), (3, 100, 12, 7), (5, 31, 11, 8)])
@pytest.mark.parametrize("wall", [False, True])
def test_node_kernels_equal_march_and_oracle(N, nx, ny, nz, wall):
    steps = 12
    w = W.random_smooth3d(N, nx, ny, nz, seed=810 + nx + wall, wall_z=wall, accept=oracle_accepts)
    print(f"case node kernels N={N} {nx}x{ny}x{nz} wall={wall} steps={steps}", flush=True)
    o = OracleSim3D(**w.params())
    o.init(w.c, w.u)
    o.step(steps)
    for precision in (64, 32):
        march = _macro(w, precision, steps, "4")
        got = _macro(w, precision, steps, "0")
        assert all(np.array_equal(a, b) for a, b in zip(got, march)), precision
        if precision == 64:
            assert max(maxabs(a, b) for a, b in zip(got, o.macro())) < 1e-10


def test_node_kernels_equal_march_beyond_the_cache():
    # N = 5 FP64, 110 x 60 x 50: 428 MB in both copies of the state
    w = W.random_smooth3d(5, 110, 60, 50, seed=823, wall_z=True, accept=oracle_accepts)
    print("case node kernels N=5 110x60x50 fp64 steps=6", flush=True)
    got, march = _macro(w, 64, 6, "0"), _macro(w, 64, 6, "4")
    assert all(np.array_equal(a, b) for a, b in zip(got, march))


@pytest.mark.parametrize("N,nx,ny,nz", [(2, 128, 7, 4), (3, 129, 5, 4), (4, 16, 5, 6), (5, 113, 9, 4),
                                        (3, 112, 13, 5), (2, 48, 4, 9)])
@pytest.mark.parametrize("wall", [False, True])
def test_row_copies_equal_march(N, nx, ny, nz, wall):
    """Stencils formed from rows copied to LDS: the longest rows that are
    copied and the first that are not, fewer rows than a workgroup holds, a
    last workgroup of one row.  Bitwise, as above."""
    w = W.random_smooth3d(N, nx, ny, nz, seed=840 + nx + wall, wall_z=wall, accept=oracle_accepts)
    print(f"case row copies N={N} {nx}x{ny}x{nz} wall={wall}", flush=True)
    for precision in (64, 32):
        got, march = _macro(w, precision, 7, "0"), _macro(w, precision, 7, "4")
        assert all(np.array_equal(a, b) for a, b in zip(got, march)), precision
