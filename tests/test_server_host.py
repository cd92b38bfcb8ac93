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
