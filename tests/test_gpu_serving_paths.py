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
