"""The serving form where a session's commands follow one another closely, over
several workgroups."""
import time

import numpy as np
import pytest

from workloads import Request, make_instance, make_requests

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


def _mixed(k, count, seed, n_hi=12):
    """A queue of requests of two to n_hi containers, some with demands no
    server has."""
    rng = np.random.default_rng([seed, k])
    inst = make_instance(k, 32, 256, 40000, 100000, 100000, background=0.7, rng=rng)
    return inst, make_requests(count, rng, 2, n_hi)


def _run(s, reqs):
    ids = [s.submit(r) for r in reqs]
    res = {r.req_id: r for r in s.drain()}
    return [res[i] for i in ids]


def _same(a, b):
    for x, y in zip(a, b, strict=True):
        assert (x.status, x.failed_at) == (y.status, y.failed_at)
        np.testing.assert_array_equal(x.hosts, y.hosts)
        np.testing.assert_array_equal(x.scores.view(np.uint32), y.scores.view(np.uint32))


@pytest.mark.parametrize("k", [32, 48])
def test_serving_idles_leaves_and_takes_commands_again(k):
    """The kernel leaves after its second without a command, the fetching
    workgroup handing out the stop; the next command starts it again at the
    ring's position, with the rounds and the state as they were.  Three times,
    with departures after each, against the plain form."""
    inst, reqs = _mixed(k, 18, seed=3)
    s = dc.Scheduler([inst], mode=dc.DC_MODE_SERVING)
    p = dc.Scheduler([inst], grid=1)
    for part in range(3):
        mine = reqs[6 * part:6 * part + 6]
        got = _run(s, mine)
        for r in mine:
            p.submit(r)
        want = p.schedule()
        _same(got, want)
        for x, y in zip(got, want):
            if x.status == 1 and x.req_id % 2 == 0:
                assert s.release(x.req_id) == dc.DC_OK and p.release(y.req_id) == dc.DC_OK
        s.drain()
        np.testing.assert_array_equal(s.state(0), p.state(0))
        time.sleep(1.5)
    s.close()
    p.close()


C5 = (dc.DC_CRIT_CPU, dc.DC_CRIT_RAM, dc.DC_CRIT_UPLINK, dc.DC_CRIT_PATHBW, dc.DC_CRIT_HOPS)


@pytest.mark.parametrize("k,crit,n_hi", [
    (34, None, 24), (38, None, 24), (44, C5, 12),      # the kernel for any k, on the default criteria and on others
    (50, None, 24), (56, C5, 8), (64, None, 8),        # pods past the pairwise commit's registers
])
@pytest.mark.parametrize("routing", [0, 1])
def test_large_data_centers_on_every_form(k, crit, n_hi, routing):
    """The automatic serving form and the automatic queue (a workgroup per pod
    each) against one workgroup per step, at sizes with no kernel of their
    own."""
    inst, reqs = _mixed(k, 8, seed=7, n_hi=n_hi)
    kw = dict(routing=routing)
    if crit is not None:
        kw.update(crit=crit, cost=(0, 0, 0, 0, 1))
    out = []
    for more in (dict(mode=dc.DC_MODE_SERVING), dict(), dict(grid=1)):
        s = dc.Scheduler([inst], **kw, **more)
        if "mode" in more:
            res = _run(s, reqs)
        else:
            for r in reqs:
                s.submit(r)
            res = s.schedule()
            assert (s.last_timing()[1] == 1) == (more == {})
        out.append((res, s.state(0)))
        s.close()
    for res, state in out[:2]:
        _same(res, out[2][0])
        np.testing.assert_array_equal(state, out[2][1])
