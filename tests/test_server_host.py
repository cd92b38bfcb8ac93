"""The server's host logic over the stand-in GPU of tests/host_double, where a
result is the number of steps its request has taken."""
import pytest

import host_util as H


def _drain(s):
    for _ in range(100):
        rc, active = s.pump()
        assert rc == 0
        if not active:
            return
    raise AssertionError("the server does not finish")


@pytest.mark.parametrize("call,nth,quantum", [
    ("launch_geom_step", 1, 4), ("launch_geom_step", 6, 4), ("hipEventRecord", 2, 4),
    ("hipStreamWaitEvent", 1, 4), ("hipStreamWaitEvent", 4, 4), ("launch_geom_step", 8, 5)])
def test_a_quantum_that_breaks_off_fails_its_requests(call, nth, quantum):
    """Three groups side by side, one of whose launches, event records or
    waits fails: the requests fail with that error, their work is waited for
    before their memory is freed, and the server goes on with others."""
    s = H.Server(quantum=quantum)
    ts = [s.submit(N, 64, 40, 11) for N in (2, 3, 4)]
    s.L.double_fail(call.encode(), nth)
    rc, _ = s.pump()
    assert rc == -4
    assert [s.poll(t) for t in ts] == [3, 3, 3]
    assert [s.result(t) for t in ts] == [-4, -4, -4]
    ts = [s.submit(N, 64, 40, steps) for N, steps in ((2, 11), (3, 3), (4, 8))]
    _drain(s)
    assert [s.result(t) for t in ts] == [11, 3, 8]
    s.close()
    assert s.L.double_unsafe() == 0


@pytest.mark.parametrize("call", ["launch_progress", "hipStreamBeginCapture", "launch_geom_step",
                                  "hipStreamEndCapture", "hipGraphInstantiate",
                                  "hipGraphLaunch"])
def test_an_error_before_a_captured_quantum_loses_no_request(call):
    """The second quantum of a resident set is captured and launched as a
    graph: an error up to its launch leaves the requests where they were."""
    s = H.Server(quantum=4)
    ts = [s.submit(N, 64, 40, 11) for N in (2, 3)]
    assert s.pump() == (0, 2)
    s.L.double_fail(call.encode(), 1)
    rc, _ = s.pump()
    assert rc == -4 and [s.poll(t) for t in ts] == [1, 1]
    _drain(s)
    assert [s.result(t) for t in ts] == [11, 11]
    s.close()
    assert s.L.double_unsafe() == 0


def test_destroyed_with_work_in_flight():
    """Requests still resident when the server is destroyed."""
    s = H.Server(quantum=3)
    for N in (2, 3, 4):
        s.submit(N, 64, 40, 100)
    assert s.pump() == (0, 3) and s.pump() == (0, 3)
    s.close()
    assert s.L.double_unsafe() == 0


def test_domains_beyond_the_cache_share_their_launches():
    """Domains whose state alone exceeds the 256 MB cache (three of 288 MB of
    one kind, one of another) run in one wave, those of one kind in one
    launch; those that fit are packed into launches that fit, in waves."""
    s = H.Server(quantum=2)
    big = [s.submit(5, 600, 600, 5, 64) for _ in range(3)] + [s.submit(3, 800, 800, 4, 64)]
    fit = [s.submit(4, 400, 400, 3, 64) for _ in range(3)] + [s.submit(2, 64, 64, 6, 32)]
    assert s.pump() == (0, 8)
    rows = [(N, ty, domains) for N, prec, ty, domains, graph, stream in H.launches()]
    assert rows.count((5, 0, 3)) == 2 and rows.count((3, 0, 1)) == 2
    assert (5, 0, 1) not in rows
    # 102 MB each: two in one launch, the third in another
    assert rows.count((4, 8, 2)) == 2 and rows.count((4, 8, 1)) == 2
    # the launches beyond the cache come last, on two streams
    last = H.launches()[-4:]
    assert {r[0] for r in last} == {3, 5} and len({r[5] for r in last}) == 2
    _drain(s)
    assert [s.result(t) for t in big + fit] == [5, 5, 5, 4, 3, 3, 3, 6]
    s.close()
    assert s.L.double_unsafe() == 0


def test_more_slots_than_one_progress_launch():
    """Resident requests on both sides of slot 256, of different step counts:
    each takes its own, over quanta that end in odd and even steps."""
    s = H.Server(slots=600, quantum=3)
    steps = [1 + (7 * i) % 11 for i in range(530)]
    ts = [s.submit(2 + i % 2, 4 + i % 5, 8, n) for i, n in enumerate(steps)]
    _drain(s)
    assert [s.result(t) for t in ts] == steps
    s.close()
