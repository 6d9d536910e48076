"""The plain form's queue kernels: a whole queue in one launch, against the
cooperative step (one launch per container step, grid = 2), bit for bit, at
the sizes where the resident kernel's layout changes."""
import numpy as np
import pytest

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
