"""Field arrays between host and device: read-backs above the size at which
several threads move chunks (8 MiB) against the initial fields and against
the checkpoint, from two domains on two threads at once; and the check of
the initial fractions, which names the first node in error wherever it lies
(one and several threads, a last block that is not full)."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _domain(nx, ny, N=3):
    import paper_1904_12553_amd as P
    import workloads as W
    return P.Domain(precision=64, N=N, nx=nx, ny=ny, sigma=W.uniform_sigma(N, 1e-3),
                    rho=np.ones(N), mu=np.full(N, 0.1))


def _fields(nx, ny, N, seed):
    r = np.random.default_rng(seed).uniform(0.1, 1.0, (N, ny, nx))
    c = r / r.sum(axis=0)
    c[-1] = 1.0 - c[:-1].sum(axis=0)
    return c


def test_large_readbacks_from_two_threads():
    got, errs = {}, []

    def work(i):
        try:
            c = _fields(1031, 900 + i, 3, i)
            d = _domain(1031, 900 + i)
            d.set_fields(c)
            s0, t0 = d.get_state()
            for _ in range(3):
                out = d.get_c()
                assert np.max(np.abs(out - c)) < 1e-13  # phi and back: a few roundings
            d.step(4)
            a = d.macro()
            d.set_state(s0, t0)
            d.step(4)
            b = d.macro()
            got[i] = all(np.array_equal(x, y) for x, y in zip(a, b))
            d.close()
        except Exception as e:  # surfaced below
            errs.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errs, errs
    assert got == {0: True, 1: True}


@pytest.mark.parametrize("nx,ny", [(40, 30), (1501, 1013)])
def test_first_node_in_error(nx, ny):
    import paper_1904_12553_amd as P
    d = _domain(nx, ny)
    good = _fields(nx, ny, 3, 7)
    d.set_fields(good)
    ref = d.get_c()
    n = nx * ny
    for bad in ([n - 1], [n // 2, n - 1], [0, n // 3], [2047 % n, 2048 % n]):
        c = good.copy().reshape(3, -1)
        for b in bad:
            c[1, b] += 1e-6
        with pytest.raises(P.NplbmError, match=rf"at node {min(bad)} \(must be 1\)"):
            d.set_fields(c)
        c[2, bad[-1]] = np.nan
        first = min(bad)
        want = rf"not finite at node {first}" if first == bad[-1] else rf"at node {first} \(must"
        with pytest.raises(P.NplbmError, match=want):
            d.set_fields(c)
    c = good.copy()
    c[0, 0, 0], c[1, 0, 0] = np.inf, -np.inf
    with pytest.raises(P.NplbmError, match="not finite at node 0"):
        d.set_fields(c)
    u = np.zeros((2, ny, nx))
    u[1, ny - 1, nx - 1] = np.nan
    with pytest.raises(P.NplbmError, match="u is not finite"):
        d.set_fields(good, u)
    assert np.array_equal(d.get_c(), ref)
    d.close()


def test_chunked_readbacks_from_two_threads():
    """Arrays that several threads move in chunks (c of 59 MiB, the last chunk
    not full), read by two domains at once, against the initial fields."""
    bad = []

    def work(i):
        try:
            c = _fields(1603, 1600 + i, 3, 20 + i)
            d = _domain(1603, 1600 + i)
            d.set_fields(c)
            for _ in range(3):
                assert np.max(np.abs(d.get_c() - c)) < 1e-13
            d.close()
        except Exception as e:  # surfaced below
            bad.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad, bad
