"""The tile kernel of small 2-D lattices against the marching kernel and the
oracle.  Both kernels evaluate the same expressions per node, so after any
number of steps c, u and p are bitwise equal (NPLBM_TILE = 0 asks for the
marching kernel); in FP64 they match the oracle within 1e-10 max-abs, the
bound of every FP64 parity test.  Sizes sit where a 32 x 8 (or 32 x 4) tile
can go wrong: lattices below one tile and below the halo, one node past an
edge, one tile column (launched through the table), several XCD runs, and
the three tile counts between which the launch changes (one and two tiles
per compute unit)."""
import os

import numpy as np
import pytest

import workloads as W
from oracle.accept import oracle_accepts
from tests.gpu_util import gpu_domain, maxabs, oracle_run

pytestmark = pytest.mark.gpu
SCHEMES = {"central": {}, "mixed": {"grad_scheme": 1}, "remark1": {"force_form": 1}}


def _macro(w, precision, steps, tile, **over):
    saved = os.environ.pop("NPLBM_TILE", None)
    if tile is not None:
        os.environ["NPLBM_TILE"] = tile
    try:
        d = gpu_domain(w, precision=precision, **over)
    finally:
        os.environ.pop("NPLBM_TILE", None)
        if saved is not None:
            os.environ["NPLBM_TILE"] = saved
    d.step(steps)
    out = d.macro()
    d.close()
    return out


@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 9), (32, 8), (33, 7), (64, 17), (35, 31),
                                   (161, 130), (256, 272), (200, 520)])
@pytest.mark.parametrize("scheme", list(SCHEMES))
@pytest.mark.parametrize("N", [2, 3, 5, 8])
def test_tiles_equal_strips_and_oracle(N, scheme, nx, ny):
    steps = 15
    sig = {"sigma_range": (0.95e-3, 1.05e-3)} if N > 5 else {}
    for wall in (False, True):
        w = W.random_smooth(N, nx, ny, seed=700 + N + nx + wall, wall_y=wall,
                            accept=oracle_accepts, **sig)
        print(f"case tile N={N} {scheme} {nx}x{ny} wall={wall} steps={steps}", flush=True)
        o = oracle_run(w, steps, **SCHEMES[scheme]).macro()
        for precision in (64, 32):
            strips = _macro(w, precision, steps, "0", **SCHEMES[scheme])
            for tile in (None, "8"):
                got = _macro(w, precision, steps, tile, **SCHEMES[scheme])
                assert all(np.array_equal(a, b) for a, b in zip(got, strips)), (precision, tile)
            if precision == 64:
                assert max(maxabs(a, b) for a, b in zip(got, o)) < 1e-10


@pytest.mark.parametrize("nx,ny", [(250, 261), (400, 193), (512, 192), (20, 3001)])
@pytest.mark.parametrize("scheme", list(SCHEMES))
@pytest.mark.parametrize("N", [2, 4, 5, 8])
def test_twelve_row_tiles_equal_strips(N, scheme, nx, ny):
    """Lattices that 8-row tiles give more than one tile per compute unit and
    12-row tiles at most one (the largest exactly 256): last tiles of 9, 1,
    12 and 1 rows, ragged and whole columns, one column.  Bitwise, as above."""
    steps = 6
    sig = {"sigma_range": (0.95e-3, 1.05e-3)} if N > 5 else {}
    for wall in (False, True):
        w = W.random_smooth(N, nx, ny, seed=900 + N + nx + wall, wall_y=wall,
                            accept=oracle_accepts, **sig)
        print(f"case tall tile N={N} {scheme} {nx}x{ny} wall={wall}", flush=True)
        for precision in (64, 32):
            strips = _macro(w, precision, steps, "0", **SCHEMES[scheme])
            got = _macro(w, precision, steps, None, **SCHEMES[scheme])
            assert all(np.array_equal(a, b) for a, b in zip(got, strips)), precision


@pytest.mark.parametrize("scheme", list(SCHEMES))
@pytest.mark.parametrize("N", [6, 7, 8])
def test_shared_collisions_equal_strips(N, scheme):
    """Many phases, whose two threads per node share the collision: one 8-row
    tile per compute unit, two, and more than are resident (256, 506 and 546
    tiles); and 4-row tiles, 255 of them.  Bitwise, as above."""
    for nx, ny in ((256, 253), (352, 366), (416, 333), (480, 68)):
        w = W.random_smooth(N, nx, ny, seed=960 + N + nx, wall_y=True, accept=oracle_accepts,
                            sigma_range=(0.95e-3, 1.05e-3))
        print(f"case shared N={N} {scheme} {nx}x{ny}", flush=True)
        for precision in (64, 32):
            strips = _macro(w, precision, 5, "0", **SCHEMES[scheme])
            got = _macro(w, precision, 5, None, **SCHEMES[scheme])
            assert all(np.array_equal(a, b) for a, b in zip(got, strips)), (nx, precision)


@pytest.mark.parametrize("N,scheme,precision,nx,ny", [
    (7, "central", 32, 800, 640), (6, "mixed", 32, 901, 650), (8, "remark1", 32, 900, 980),
    (6, "remark1", 64, 560, 520), (8, "central", 64, 777, 700)])
def test_tiles_beyond_the_cache_equal_strips(N, scheme, precision, nx, ny):
    """Many phases, which are stepped by tiles beyond 256 MB of state (287 to
    713 MB).  Bitwise, as above."""
    w = W.random_smooth(N, nx, ny, seed=980 + N + nx, accept=oracle_accepts,
                        sigma_range=(0.95e-3, 1.05e-3))
    print(f"case big tile N={N} {scheme} fp{precision} {nx}x{ny}", flush=True)
    strips = _macro(w, precision, 3, "0", **SCHEMES[scheme])
    got = _macro(w, precision, 3, None, **SCHEMES[scheme])
    assert all(np.array_equal(a, b) for a, b in zip(got, strips))
