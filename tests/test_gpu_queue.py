"""The plain form's queue kernels: a whole queue in one launch, against the
cooperative step (one launch per container step, grid = 2), bit for bit, at
the sizes where the resident kernel's layout changes."""
import numpy as np
import pytest

import oracle as O
from parity import lockstep
from workloads import make_instance, make_requests

pytestmark = pytest.mark.gpu

dc = pytest.importorskip("paper_1909_07673_amd")

C5 = (dc.DC_CRIT_CPU, dc.DC_CRIT_RAM, dc.DC_CRIT_UPLINK, dc.DC_CRIT_PATHBW, dc.DC_CRIT_HOPS)


def _queue(k, n_lo, n_hi, count, seed, density=0.5):
    rng = np.random.default_rng([seed, k, n_hi])
    inst = make_instance(k, 32, 256, 40000, 100000, 100000, background=0.7, rng=rng)
    reqs = make_requests(count, rng, n_lo, n_hi, density=density)
    return inst, reqs


def _schedule(inst, reqs, **kw):
    s = dc.Scheduler([inst], **kw)
    for r in reqs:
        s.submit(r)
    res = s.schedule_array()
    out = {f: np.ascontiguousarray(res[f]) for f in ("status", "n", "failed_at", "host", "score")}
    out["state"] = s.state(0)
    out["paths"] = [s.paths(int(i)) for i, ok in zip(res["req_id"], res["status"]) if ok]
    s.close()
    return out


def _same(a, b):
    for f in ("status", "n", "failed_at", "host", "state"):
        np.testing.assert_array_equal(a[f], b[f], err_msg=f)
    np.testing.assert_array_equal(a["score"].view(np.uint32), b["score"].view(np.uint32))
    assert len(a["paths"]) == len(b["paths"])
    for x, y in zip(a["paths"], b["paths"]):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("k,n_lo,n_hi,count,crit", [
    (4, 2, 6, 40, 4),       # one wavefront, 16 servers
    (6, 2, 9, 40, 5),       # 54 servers: rows not a multiple of 16 bytes
    (10, 60, 64, 12, 4),    # every pair of the largest requests staged
    (18, 2, 64, 20, 4),     # several peer chunks
    (20, 60, 64, 12, 4),    # pairs brought in step by step, several chunks
    (20, 2, 8, 30, 5),      # small requests: no accumulator rows
    (22, 2, 12, 20, 4),     # beyond the resident layout
])
@pytest.mark.parametrize("routing", [0, 1])
def test_queue_matches_cooperative_step(k, n_lo, n_hi, count, crit, routing):
    inst, reqs = _queue(k, n_lo, n_hi, count, seed=11, density=0.9 if n_lo >= 60 else 0.5)
    kw = dict(routing=routing)
    if crit == 5:
        kw.update(crit=C5, cost=(0, 0, 0, 0, 1))
    a, b = _schedule(inst, reqs, **kw), _schedule(inst, reqs, grid=2, **kw)
    _same(a, b)
    assert a["n"].max() >= n_hi - 4


@pytest.mark.parametrize("block", [64, 256, 512, 1024])
def test_queue_block_sizes(block):
    inst, reqs = _queue(12, 2, 24, 20, seed=5)
    _same(_schedule(inst, reqs, block=block), _schedule(inst, reqs, grid=2))


def test_queue_several_instances():
    """Instances of one plain context: each its own workgroup, as if alone."""
    qs = [_queue(8, 2, 16, 12, seed=s) for s in range(5)]
    s = dc.Scheduler([i for i, _ in qs])
    for r in range(12):
        for x, (_, reqs) in enumerate(qs):
            s.submit(reqs[r], instance=x)
    res = s.schedule_array()
    for x, (inst, reqs) in enumerate(qs):
        one = _schedule(inst, reqs)
        mine = res[res["instance"] == x]
        for f in ("status", "n", "failed_at", "host"):
            np.testing.assert_array_equal(mine[f], one[f])
        np.testing.assert_array_equal(mine["score"].view(np.uint32), one["score"].view(np.uint32))
        np.testing.assert_array_equal(s.state(x), one["state"])
    s.close()


def _ahp(inst, reqs, crit=None, cost=None, **kw):
    if crit is not None:
        kw.update(crit=crit, cost=cost)
    return _schedule(inst, reqs, method=dc.DC_AHP, **kw)


C8 = (0, 1, 2, 3, 4, 5, 0, 4)


@pytest.mark.parametrize("k,n_lo,n_hi,count,crit,cost", [
    (4, 2, 6, 40, None, None),
    (4, 2, 6, 20, C8, (0, 0, 0, 0, 0, 1, 1, 1)),    # more workgroups than pods
    (6, 60, 64, 6, C5, (0, 0, 0, 0, 1)),
    (16, 2, 24, 20, None, None),                     # 1,024 servers: one per thread
    (18, 2, 24, 12, C5, (1, 0, 1, 0, 1)),
    (20, 4, 4, 24, None, None),
    (24, 2, 24, 8, C5, (0, 0, 0, 0, 1)),             # 3,456: column sums shared out, 512 threads
    (26, 2, 24, 8, None, None),                      # 4,394: 1,024 threads
    (30, 2, 32, 6, (4,), (0,)),                      # one criterion, 30 slices
    (32, 8, 64, 6, C5, (0, 0, 0, 0, 1)),             # the largest
])
@pytest.mark.parametrize("routing", [0, 1])
def test_ahp_queue_matches_launches(k, n_lo, n_hi, count, crit, cost, routing):
    """One launch, its column sums from counts, against the sorted passes of
    one launch per stage (grid = 1): the same sums up to FP64 rounding, so
    the same FP32 scores."""
    inst, reqs = _queue(k, n_lo, n_hi, count, seed=3)
    _same(_ahp(inst, reqs, crit, cost, routing=routing), _ahp(inst, reqs, crit, cost, routing=routing, grid=1))


@pytest.mark.parametrize("cap", [0, 1, 43000, 100000])
def test_ahp_queue_capacities(cap):
    """Capacities at the ends of the position table's range, and past it."""
    rng = np.random.default_rng(cap)
    inst = make_instance(16, 32, 256, cap, 100000, 100000, background=0.7, rng=rng)
    reqs = make_requests(12, rng, 1, 12, bw_lo=1, bw_hi=max(1, cap // 20))
    _same(_ahp(inst, reqs, C5, (0, 0, 0, 0, 1)), _ahp(inst, reqs, C5, (0, 0, 0, 0, 1), grid=1))


@pytest.mark.parametrize("k,method", [(16, dc.DC_AHP), (24, dc.DC_TOPSIS)])
def test_queue_that_cannot_start_runs_step_by_step(k, method):
    """With 1 us for its workgroups to meet, a queue kernel that finds them
    late leaves everything alone, and the queue runs launch by launch: the
    same results either way, again and again."""
    inst, reqs = _queue(k, 2, 12, 8, seed=9)
    want = _schedule(inst, reqs, method=method, grid=1)
    s = dc.Scheduler([inst], method=method, grid_timeout_us=1)
    for r in reqs:
        s.submit(r)
    for _ in range(3):
        s.rewind()
        res = s.schedule_array()
        for f in ("status", "n", "failed_at", "host"):
            np.testing.assert_array_equal(res[f], want[f])
        np.testing.assert_array_equal(res["score"].view(np.uint32), want["score"].view(np.uint32))
        np.testing.assert_array_equal(s.state(0), want["state"])
    s.close()


def test_topsis_queue_two_calls_and_releases():
    """Several schedule calls with departures between them on one context:
    rounds and tags go on from one launch to the next."""
    inst, reqs = _queue(24, 2, 16, 16, seed=21)
    out = []
    for grid in (0, 2):
        s = dc.Scheduler([inst], grid=grid)
        got = []
        for lo in range(0, 16, 4):
            ids = [s.submit(r) for r in reqs[lo:lo + 4]]
            res = s.schedule_array()
            got.append(res.copy())
            for i, ok in zip(ids, res["status"]):
                if ok and i % 2 == 0:
                    assert s.release(i) == dc.DC_OK
        out.append((got, s.state(0)))
        s.close()
    for a, b in zip(out[0][0], out[1][0]):
        for f in ("status", "failed_at", "host"):
            np.testing.assert_array_equal(a[f], b[f])
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("k,up,cost", [
    (34, 40000, (0, 0, 0, 0, 1)),      # 9,826 servers: a chunk of 98 columns with a tail of two
    (36, 1000, (1, 1, 1, 1, 0)),       # 11,664: few distinct values, other directions
    (48, 40000, (0, 0, 0, 0, 1)),      # 27,648
    (34, 90000, (0, 0, 0, 0, 1)),      # past the counting kernel: the pairwise passes on both sides
])
def test_ahp_large_matches_pairwise(k, up, cost):
    """Row sums by distinct value against the pairwise passes (grid = 1): the
    same FP32 terms in the same order, so every score vector is the same bit
    for bit."""
    rng = np.random.default_rng([k, up])
    inst = make_instance(k, 32, 256, up, 100000, 100000, background=0.99 if up == 1000 else 0.7, rng=rng)
    reqs = make_requests(2, rng, 4, 8, bw_lo=1, bw_hi=up // 20)
    out = []
    for grid in (0, 1):
        s = dc.Scheduler([inst], method=dc.DC_AHP, crit=C5, cost=cost, grid=grid, trace_stride=1, trace_cap=16)
        for r in reqs:
            s.submit(r)
        res = s.schedule_array()
        meta, scores = s.trace()
        out.append((res.copy(), meta, scores.view(np.uint32).copy(), s.state(0)))
        s.close()
    (a, ma, sa, ta), (b, mb, sb, tb) = out
    np.testing.assert_array_equal(ma, mb)
    assert len(ma) >= 4
    np.testing.assert_array_equal(sa, sb)
    for f in ("status", "failed_at", "host"):
        np.testing.assert_array_equal(a[f], b[f])
    np.testing.assert_array_equal(ta, tb)


# data centers of 8,192 servers whose residual CPU draws (numpy's generator of
# this seed, uniform over 0..40,000; cost says which way it counts) have a row
# sum near the middle of two FP32 values: found on the CPU as those where prefix
# sums taken in another order of FP64 additions round it to the other one
ROUNDING_SEEDS = [(37977, 1), (55437, 1), (57282, 1), (69294, 1), (82920, 0), (90644, 1), (96662, 1), (107159, 1)]


@pytest.mark.parametrize("seed,cost", ROUNDING_SEEDS)
def test_ahp_score_bits_on_every_path(seed, cost):
    """One launch for the queue and one launch per stage (which the first falls
    back to when its workgroups cannot meet) add the same FP64 terms in the same
    order: every score of the step is the same bit for bit."""
    cpu = np.random.default_rng(seed).integers(0, 40001, 8192).astype(np.int32)
    inst = make_instance(32, 40000, 256, 40000, 100000, 100000, background=0.0, rng=np.random.default_rng(0))
    inst.host_used = np.stack([40000 - cpu, np.zeros_like(cpu)])
    req = make_requests(1, np.random.default_rng(1), 1, 1)[0]
    out = []
    for grid in (0, 1):
        s = dc.Scheduler([inst], method=dc.DC_AHP, crit=(dc.DC_CRIT_CPU,), cost=(cost,), grid=grid, trace_stride=1,
                         trace_cap=4)
        s.submit(req)
        res = s.schedule_array()
        assert (s.last_timing()[1] == 1) == (grid == 0)
        out.append((s.trace()[1].view(np.uint32).copy(), res["host"].copy(), s.state(0)))
        s.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_topsis_queue_after_65535_rounds_without_outcome():
    """A request that is placed, 65,535 that find no server (one round each,
    none with an outcome), then requests that are placed again: the outcome the
    workgroups waited for last is 65,536 rounds old, and must not be taken for
    the next one.  As if the requests between had not been there."""
    inst, reqs = _queue(22, 6, 12, 6, seed=33)
    none = make_requests(1, np.random.default_rng(1), 1, 1)[0]
    none.cpu = np.full(1, 33, np.int32)                  # one core more than a server has
    want = _schedule(inst, reqs, grid=1)
    assert want["status"][0] == 1 and want["status"][1:].sum() >= 2
    s = dc.Scheduler([inst])
    s.submit(reqs[0])
    for _ in range(65535):
        s.submit(none)
    for r in reqs[1:]:
        s.submit(r)
    res = s.schedule_array()
    assert s.last_timing()[1] == 1                        # one launch for all of them
    assert not res["status"][1:65536].any() and not res["failed_at"][1:65536].any()
    mine = res[[0, *range(65536, len(res))]]
    for f in ("status", "n", "failed_at", "host"):
        np.testing.assert_array_equal(mine[f], want[f])
    np.testing.assert_array_equal(mine["score"].view(np.uint32), want["score"].view(np.uint32))
    np.testing.assert_array_equal(s.state(0), want["state"])
    s.close()


@pytest.mark.parametrize("k,crit,cost,one", [
    (20, C8, (0, 0, 0, 0, 0, 1, 1, 1), False),      # eight criteria: the state does not fit one workgroup
    (22, None, None, True),
    (26, C5, (0, 0, 0, 0, 1), False),
    (28, C5, (0, 0, 0, 0, 1), True),
])
def test_topsis_queue_where_it_is_faster(k, crit, cost, one):
    """Beyond one workgroup's LDS a queue runs in one launch on the default
    criteria at any size, on others from k = 28 on, and step by step below;
    the same results as the cooperative steps."""
    inst, reqs = _queue(k, 2, 12, 8, seed=41)
    kw = {} if crit is None else dict(crit=crit, cost=cost)
    s = dc.Scheduler([inst], **kw)
    for r in reqs:
        s.submit(r)
    s.schedule_array()
    launches, steps = s.last_timing()[1:]
    assert launches == (1 if one else steps)
    s.close()
    _same(_schedule(inst, reqs, **kw), _schedule(inst, reqs, grid=2, **kw))


@pytest.mark.parametrize("k,method", [(48, dc.DC_TOPSIS), (32, dc.DC_AHP)])
def test_refused_start_runs_launch_by_launch(k, method):
    """1 us is less than this many workgroups need to meet (measured: twenty of
    twenty starts refused): the launch count shows the steps that ran after the
    refused start, and the results are those of the queue kernel."""
    inst, reqs = _queue(k, 2, 6, 4, seed=17)
    want = _schedule(inst, reqs, method=method)
    s = dc.Scheduler([inst], method=method, grid_timeout_us=1)
    for r in reqs:
        s.submit(r)
    refused = 0
    for _ in range(5):
        s.rewind()
        res = s.schedule_array()
        launches, steps = s.last_timing()[1:]
        assert launches == 1 or launches >= 1 + steps
        refused += launches > 1
        for f in ("status", "n", "failed_at", "host"):
            np.testing.assert_array_equal(res[f], want[f])
        np.testing.assert_array_equal(res["score"].view(np.uint32), want["score"].view(np.uint32))
        np.testing.assert_array_equal(s.state(0), want["state"])
    s.close()
    assert refused >= 1


@pytest.mark.parametrize("k,up,launches", [(16, 100000, 6), (34, 90000, 5)])
def test_ahp_past_the_counting_kernels_against_the_oracle(k, up, launches):
    """Capacities whose position table does not fit LDS (up to 8,192 servers the
    sorted passes, beyond the pairwise ones): several launches per step, in
    lockstep with the oracle."""
    rng = np.random.default_rng([k, up])
    inst = make_instance(k, 32, 256, up, 100000, 100000, background=0.7, rng=rng)
    reqs = make_requests(1, rng, 3, 3, bw_lo=1, bw_hi=up // 20)
    s = dc.Scheduler([inst], method=dc.DC_AHP, crit=C5, cost=(0, 0, 0, 0, 1), trace_stride=1, trace_cap=8)
    ids = [s.submit(r) for r in reqs]
    res = {r.req_id: r for r in s.schedule()}
    n, steps = s.last_timing()[1:]
    assert n >= launches * steps
    o = O.Oracle(inst, O.method(kind=O.AHP, crit=(O.CRIT_CPU, O.CRIT_RAM, O.CRIT_UPLINK, O.CRIT_PATHBW, O.CRIT_HOPS),
                                cost=(0, 0, 0, 0, 1)))
    lockstep(o, s, ids, reqs, res, check_paths=True)
    s.close()


@pytest.mark.parametrize("k,method", [(24, dc.DC_TOPSIS), (16, dc.DC_AHP)])
def test_autotune_times_the_launches_a_block_size_governs(k, method):
    """A context whose queue runs in one launch over several workgroups takes no
    block size there: what is timed is the launch-by-launch form."""
    inst, reqs = _queue(k, 2, 6, 4, seed=19)
    s = dc.Scheduler([inst], method=method)
    for r in reqs:
        s.submit(r)
    t = s.autotune_cached()
    _, launches, steps = s.last_timing()
    assert t["candidates"] == 3 and launches >= steps >= 6 * sum(len(r.cpu) for r in reqs)
    s.schedule_array()
    assert s.last_timing()[1] == 1                        # the queue itself as before
    s.close()


def test_autotune_of_a_cooperative_context():
    """The cooperative step has a block size of its own: what is timed is the
    form over one workgroup (one launch per pass: three sizes, twice each),
    whose entry other contexts of the size read from a cache."""
    inst, reqs = _queue(16, 2, 6, 4, seed=23)
    s = dc.Scheduler([inst], grid=2)
    for r in reqs:
        s.submit(r)
    t = s.autotune_cached()
    assert t["candidates"] == 3 and s.last_timing()[1] == 6
    s.schedule_array()
    assert s.last_timing()[1] >= sum(len(r.cpu) for r in reqs)        # its own launches as before
    s.close()
