"""The serving form where a session's commands follow one another closely, over
several workgroups."""
import numpy as np
import pytest

from workloads import Request, make_instance

pytestmark = pytest.mark.gpu

dc = pytest.importorskip("paper_1909_07673_amd")


@pytest.mark.parametrize("k,grid", [(32, 0), (8, 2)])
def test_serving_departures_seen_by_the_next_request(k, grid):
    """A request that fills a data center, its departure and the same request
    again, 40 times with both commands in flight together: every time it finds
    all that the departure gave back, on every workgroup, so it is placed as the
    first time, and at the end nothing is held."""
    n = 64
    inst = make_instance(k, 8, 64, 40000, 40000, 40000)
    rng = np.random.default_rng(k)
    edges = np.array([(i, j, 600) for j in range(1, n) for i in range(j) if rng.random() < 0.3 or i == j - 1], np.int32)
    big = Request(cpu=np.full(n, 5, np.int32), ram=np.full(n, 5, np.int32), edges=edges)
    s = dc.Scheduler([inst], mode=dc.DC_MODE_SERVING, grid=grid)
    start = s.state(0)
    first = None
    rid = s.submit(big)
    for _ in range(40):
        got = {r.req_id: r for r in s.drain()}[rid]
        assert got.status == 1
        first = first or got
        np.testing.assert_array_equal(got.hosts, first.hosts)
        np.testing.assert_array_equal(got.scores.view(np.uint32), first.scores.view(np.uint32))
        assert s.release(rid) == dc.DC_OK
        rid = s.submit(big)
    s.drain()
    assert s.release(rid) == dc.DC_OK
    s.drain()
    np.testing.assert_array_equal(s.state(0), start)
    s.close()


def test_service_latency_covers_bringing_the_request_in():
    """The service latency of a request that finds the kernel idle covers its
    way from host memory (at least three reads of a microsecond, one after
    another: sequence number, fields, request); of one that waits behind
    another, that way has passed meanwhile."""
    inst = make_instance(32, 32, 256, 40000, 40000, 40000)
    none = Request(cpu=np.full(1, 33, np.int32), ram=np.full(1, 1, np.int32), edges=np.zeros((0, 3), np.int32))
    n = 32
    edges = np.array([(i, j, 100) for j in range(1, n) for i in range(j)], np.int32)
    long = Request(cpu=np.full(n, 1, np.int32), ram=np.full(n, 1, np.int32), edges=edges)
    s = dc.Scheduler([inst], mode=dc.DC_MODE_SERVING)
    for _ in range(20):
        s.submit(none)
        s.drain()
    lone = s.latency_us()
    for _ in range(10):
        s.submit(long)
        s.submit(none)
        s.submit(none)
        s.drain()
    queued = s.latency_us()[20:].reshape(10, 3)[:, 1:]
    s.close()
    assert np.median(lone) >= np.median(queued) + 3.0, (np.median(lone), np.median(queued))
