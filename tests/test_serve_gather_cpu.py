"""When a server without the lone path holds jobs back for others to join (host
logic, no GPU): never by default, and with gather_ms only while it can pay."""
import inspect
import types

import pytest


def _serve():
    pytest.importorskip("torch")
    from paper_1107_4543_amd import serve
    return serve


def job(arrival):
    return types.SimpleNamespace(arrival=arrival)


def until(gather_s, queue, pending, active, now, max_members=4):
    srv = types.SimpleNamespace(gather_s=gather_s, max_members=max_members)
    return _serve().Server._gather_until(srv, queue, pending, active, now)


def test_a_server_does_not_wait_by_default():
    assert inspect.signature(_serve().Server).parameters["gather_ms"].default == 0
    assert until(0.0, [job(1.0)], [job(1.0001)], {}, 1.0) is None


def test_jobs_gather_only_while_it_can_pay():
    first, second, later = job(1.0), job(1.0004), job(2.0)
    # an empty server, jobs to come: until 1 ms after the first one's arrival,
    # whatever the order of the queue
    assert until(1e-3, [first], [later], {}, 1.0) == pytest.approx(1.001)
    assert until(1e-3, [second, first], [later], {}, 1.0005) == pytest.approx(1.001)
    assert until(1e-3, [first], [later], {}, 1.001) is None          # the time has passed
    assert until(1e-3, [first], [later], {1: first}, 1.0) is None    # jobs run already
    assert until(1e-3, [first], [], {}, 1.0) is None                 # the last job
    assert until(1e-3, [], [later], {}, 1.0) is None                 # nothing to hold back
    assert until(1e-3, [first, second], [later], {}, 1.0005, max_members=2) is None   # the members are filled
