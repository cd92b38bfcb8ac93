"""Served sets that do not fit the 256 MB Infinity Cache, and more resident
requests than one progress launch takes: every result is bitwise that of the
request alone."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _serve(jobs, **server):
    import paper_1904_12553_amd as P
    srv = P.Server(**server)
    tickets = [srv.submit(w.c, w.u, nsteps=steps, precision=prec, **w.params())
               for w, prec, steps in jobs]
    for _ in range(1000):
        if srv.pump() == 0:
            break
    out = [srv.result(t)[:3] for t in tickets]
    srv.close()
    return out


def _alone(w, prec, steps):
    import paper_1904_12553_amd as P
    d = P.Domain(precision=prec, **w.params())
    d.set_fields(w.c, w.u)
    d.step(steps)
    out = d.macro()
    d.close()
    return out


def test_domains_beyond_the_cache_in_a_mix():
    """Two marched domains of one launch (276 MB each), two groups of tiles in
    two waves (198 and 155 MB) and a small one beside them; quanta of 5 steps,
    the first as it stands, the others captured until a request finishes."""
    import paper_1904_12553_amd as P
    mk = lambda N, nx, ny, seed, wall: W.random_smooth(N, nx, ny, seed=seed, wall_y=wall,
                                                       accept=P.accepts)
    jobs = [(mk(3, 752, 750, 1201, True), 64, 23), (mk(3, 750, 752, 1202, False), 64, 12),
            (mk(5, 700, 700, 1203, True), 32, 17), (mk(3, 897, 700, 1204, False), 32, 21),
            (mk(3, 40, 30, 1205, False), 32, 9)]
    print("case served beyond the cache: " + ", ".join(
        f"N={w.N} {w.nx}x{w.ny} fp{p} {s}" for w, p, s in jobs), flush=True)
    served = _serve(jobs, hbm_budget=8 << 30, max_slots=8, quantum=5)
    for got, (w, prec, steps) in zip(served, jobs):
        want = _alone(w, prec, steps)
        assert all(np.array_equal(a, b) for a, b in zip(got, want)), (w.N, w.nx, w.ny)


def test_more_than_256_resident_requests():
    """300 small requests resident at once, 1 to 11 steps in quanta of 3."""
    import paper_1904_12553_amd as P
    kinds = [W.random_smooth(N, nx, 8, seed=1300 + N + nx, accept=P.accepts)
             for N in (2, 3) for nx in (5, 33)]
    jobs = [(kinds[i % 4], 32, 1 + (7 * i) % 11) for i in range(300)]
    print("case 300 resident requests", flush=True)
    served = _serve(jobs, hbm_budget=8 << 30, max_slots=320, quantum=3)
    want = {}
    for i, (got, (w, prec, steps)) in enumerate(zip(served, jobs)):
        key = (i % 4, steps)
        if key not in want:
            want[key] = _alone(w, prec, steps)
        assert all(np.array_equal(a, b) for a, b in zip(got, want[key])), (i, steps)
