"""Cases of use of the scheduler and of its scoring stage, for timing.

listed() gives the fixed cases and draw() more of the same ranges; prepare()
makes what a program holds before a call (data centers, requests, contexts,
decision matrices), run() is one pass through the public entry points, work()
what the pass cannot do without, and exact() the floating-point outputs in
64 bits, computed here with numpy and torch alone.

Kinds of case:

  online   requests arrive at a running data center: submit, schedule,
           read the state (for the fragmentation shares), and the accepted
           ones depart again.  The event replay does this at every event.
  replay   a queue of requests, uploaded once, is scheduled from the start
           state, as in planning runs and parameter studies.
  batched  the same over many independent data centers in one call.
  serving  a session of the persistent form: open, a stream of requests and
           departures, close.
  tiles    the scoring stage alone, over decision matrices on the device.

Units: cores, GB, Mbps, as everywhere in this repository.
"""
import math
import types

import numpy as np
import torch

import paper_1909_07673_amd as dc

# Server CPU and RAM, then the capacity of each link level.
CAPS = {
    "even": (32, 256, 10000, 10000, 10000),        # a small rack, one link speed
    "small": (24, 256, 1000, 1000, 1000),          # the paper's evaluation, section VI-A
    "large": (32, 256, 40000, 100000, 100000),     # 40 Gbps servers, 100 Gbps fabric
}
# Demands: highest CPU, RAM, then lowest and highest bandwidth of a pair.
DEMANDS = {"even": (8, 32, 100, 2000), "small": (2, 4, 1, 50), "large": (8, 32, 100, 2000)}
BACKGROUND = {"even": 0.0, "small": 0.0, "large": 0.7}

CRIT4 = (dc.DC_CRIT_CPU, dc.DC_CRIT_RAM, dc.DC_CRIT_ACTIVE, dc.DC_CRIT_PATHBW)
CRIT5 = (dc.DC_CRIT_CPU, dc.DC_CRIT_RAM, dc.DC_CRIT_UPLINK, dc.DC_CRIT_PATHBW, dc.DC_CRIT_HOPS)

# Columns of a decision matrix: residual CPU, RAM, the placed flag, path
# bandwidth, hops (a cost), uplink bandwidth, containers placed, any value.
COLUMNS = ((0, 32), (0, 256), (0, 1), (0, 40000), (0, 384), (0, 100000), (0, 10), (0, (1 << 22) - 1))


def listed():
    return [
        # one small tenant request at a small data center: the latency of a
        # single decision, nearly all of it launches and host work
        dict(name="online_k4", kind="online", k=4, caps="even", method="topsis", crit=4, requests=1, n_lo=2, n_hi=6,
             pods=False, ranges=False, routing=0),
        # one event of the paper's evaluation: 24 arrivals of 4 containers,
        # half of them in pods, demand intervals, 2,000 servers
        dict(name="event_k20", kind="online", k=20, caps="small", method="topsis", crit=4, requests=24, n_lo=4, n_hi=4,
             pods=True, ranges=True, routing=0),
        # the same under AHP, the paper's other method
        dict(name="event_k20_ahp", kind="online", k=20, caps="small", method="ahp", crit=4, requests=24, n_lo=4,
             n_hi=4, pods=True, ranges=True, routing=0),
        # a queue of ordinary requests on one loaded data center of 1,024 servers
        dict(name="queue_k16", kind="replay", k=16, caps="large", method="topsis", crit=4, requests=500, n_lo=2,
             n_hi=32, pods=False, ranges=False, routing=0),
        # AHP with five criteria on 8,192 servers, large requests
        dict(name="queue_k32_ahp", kind="replay", k=32, caps="large", method="ahp", crit=5, requests=60, n_lo=8,
             n_hi=64, pods=False, ranges=False, routing=0),
        # AHP on the largest data center of this repository, 27,648 servers
        dict(name="queue_k48_ahp", kind="replay", k=48, caps="large", method="ahp", crit=5, requests=3, n_lo=8,
             n_hi=64, pods=False, ranges=False, routing=0),
        # many independent data centers at once, a queue each: the form with
        # the highest throughput
        dict(name="batched_256_k16", kind="batched", instances=256, k=16, caps="large", method="topsis", crit=4,
             r_lo=16, r_hi=128, n_lo=2, n_hi=48, pods=False, ranges=False, routing=0),
        # the same at an odd size, with pods, demand intervals and the
        # paper's order of routing (after a request's last container)
        dict(name="batched_100_k10", kind="batched", instances=100, k=10, caps="large", method="topsis", crit=4,
             r_lo=16, r_hi=64, n_lo=2, n_hi=24, pods=True, ranges=True, routing=1),
        # a session of the serving form on 27,648 servers: 300 requests, the
        # accepted ones departing half a stream later
        dict(name="serving_k48", kind="serving", k=48, caps="large", method="topsis", crit=4, requests=300, n_lo=2,
             n_hi=64, pods=False, ranges=False, routing=0),
        # one decision matrix of the largest data center, every score wanted
        dict(name="tiles_1_k48", kind="tiles", T=1, C=4, N=27648, feasible=True, scores=True),
        # matrices of a 2,000-server data center, five criteria, with masks,
        # every score wanted
        dict(name="tiles_2048_k20", kind="tiles", T=2048, C=5, N=2000, feasible=True, scores=True),
        # scoring at full bandwidth: 512 MiB of matrices
        dict(name="tiles_32768_k16", kind="tiles", T=32768, C=4, N=1024, feasible=False, scores=False),
    ]


def _log(rng, lo, hi):
    return min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49))))))


def draw(rng):
    most = max(c["flops"] for c in map(work, listed()))
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= most and _fits(case):
            return case


def _fits(case):
    # passes of at most some hundred milliseconds
    if case["kind"] == "tiles":
        return case["T"] * case["C"] * case["N"] <= 1 << 27 and case["T"] * case["N"] <= 1 << 26
    if case["method"] == "ahp":
        n = (case["n_lo"] + case["n_hi"]) / 2
        return case["requests"] * n <= (110 if case["k"] > 32 else 2500)
    return True


def _draw(rng):
    kind = rng.choice(["online", "online", "replay", "replay", "batched", "serving", "tiles", "tiles", "tiles"])
    if kind == "tiles":
        n = rng.choice([_log(rng, 16, 27648), rng.choice(range(4, 49, 2)) ** 3 // 4])
        return dict(kind=kind, T=_log(rng, 1, 32768), C=rng.randint(1, 8), N=n, feasible=rng.random() < 0.5,
                    scores=rng.random() < 0.4)
    opt = dict(pods=rng.random() < 0.4, ranges=rng.random() < 0.4, routing=int(rng.random() < 0.25))
    if kind == "online":
        caps, hi = rng.choice([("even", 8), ("small", 24), ("large", 24)])
        lo, up = sorted((rng.randint(2, 12), rng.randint(2, 12)))
        return dict(kind=kind, k=2 * rng.randint(2, hi // 2), caps=caps, method=rng.choice(["topsis", "topsis", "ahp"]),
                    crit=4, requests=_log(rng, 1, 48), n_lo=lo, n_hi=up, **opt)
    up = _log(rng, 8, 64)
    size = dict(caps="large", n_lo=rng.randint(2, 8), n_hi=up)
    if kind == "replay":
        if rng.random() < 0.5:
            return dict(kind=kind, k=2 * rng.randint(4, 16), method="topsis", crit=rng.choice([4, 4, 5]),
                        requests=_log(rng, 20, 500), **size, **opt)
        return dict(kind=kind, k=2 * rng.randint(8, 24), method="ahp", crit=rng.choice([4, 5]),
                    requests=_log(rng, 2, 120), **size, **opt)
    if kind == "batched":
        r = _log(rng, 8, 100)
        return dict(kind=kind, instances=_log(rng, 8, 300), k=2 * rng.randint(2, 8), method="topsis", crit=4, r_lo=r // 2,
                    r_hi=r, **size, **opt)
    return dict(kind=kind, k=2 * rng.randint(8, 24), method="topsis", crit=4, requests=_log(rng, 60, 300), **size, **opt)


# ---------------------------------------------------------------- inputs

def _instance(k, caps, rng):
    """A k-ary fat-tree, with background load where its kind has it."""
    c, b, n = CAPS[caps], BACKGROUND[caps], k ** 3 // 4
    used = [None] * 5
    if b:
        used = [np.floor(rng.uniform(0.0, b, n) * cap).astype(np.int32) for cap in c]
    return types.SimpleNamespace(k=k, host_cpu=c[0], host_ram=c[1], bw_host_edge=c[2], bw_edge_agg=c[3],
                                 bw_agg_core=c[4], host_used=np.stack(used[:2]) if b else None,
                                 link_used=np.stack(used[2:]) if b else None)


def _request(case, rng):
    """A tenant request: containers, a connected random graph of traffic
    over half of all pairs, and optionally pods and demand intervals."""
    chi, rhi, blo, bhi = DEMANDS[case["caps"]]
    n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
    cpu, ram = rng.integers(1, chi + 1, n).astype(np.int32), rng.integers(1, rhi + 1, n).astype(np.int32)
    target = max(n - 1, math.ceil(n * (n - 1) / 4))
    j = np.arange(1, n)
    i = (rng.random(n - 1) * j).astype(np.int64)                # node j joins an earlier node
    tree = np.zeros((n, n), bool)
    tree[i, j] = True
    a, b = np.nonzero(np.triu(~tree, 1))
    pick = rng.permutation(a.size)[:target - (n - 1)]
    i, j = np.concatenate([i, a[pick]]), np.concatenate([j, b[pick]])
    bw = rng.integers(blo, bhi + 1, i.size)
    req = types.SimpleNamespace(cpu=cpu, ram=ram, pod=None, cpu_max=None, ram_max=None, bw_max=None,
                                edges=np.stack([i, j, bw], 1).astype(np.int32))
    if case["pods"]:
        # up to half of the containers in pods of two to four
        g = int(rng.integers(0, n // 2 + 1))
        req.pod = np.full(n, -1, np.int32)
        who = rng.permutation(n)[:g if g > 1 else 0]
        at = pod = 0
        while who.size - at >= 2:
            s = int(rng.integers(2, 5))
            s += who.size - at - s == 1
            req.pod[who[at:at + s]] = pod
            at, pod = at + s, pod + 1
    if case["ranges"] and case["caps"] == "small":
        # the paper's bounds are the maxima
        req.cpu_max, req.ram_max, req.bw_max = cpu, ram, req.edges[:, 2].copy()
        req.cpu, req.ram = rng.integers(1, cpu + 1).astype(np.int32), rng.integers(1, ram + 1).astype(np.int32)
        req.edges[:, 2] = rng.integers(1, req.bw_max + 1)
    elif case["ranges"]:
        req.cpu_max, req.ram_max, req.bw_max = (
            (x + rng.integers(0, x + 1)).astype(np.int32) for x in (cpu, ram, req.edges[:, 2]))
    return req


def _queue(case, i):
    """Requests queued at data center i: spread evenly over [r_lo, r_hi]."""
    return case["r_lo"] + i * 7919 % case["instances"] * (case["r_hi"] - case["r_lo"] + 1) // case["instances"]


def _inputs(case, seed):
    rng = np.random.default_rng([seed, case["k"]])
    insts, reqs = [], []
    for _ in range(case.get("instances", 1)):
        insts.append(_instance(case["k"], case["caps"], rng))
        count = case["requests"] if "requests" in case else _queue(case, len(reqs))
        reqs.append([_request(case, rng) for _ in range(count)])
    return insts, reqs


def _matrices(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((case["T"], case["C"], case["N"]), dtype=torch.int32, device="cuda")
    for c in range(case["C"]):
        lo, hi = COLUMNS[c]
        x[:, c] = torch.randint(lo, hi + 1, (case["T"], case["N"]), generator=g, dtype=torch.int32, device="cuda")
    f = None
    if case["feasible"]:
        f = (torch.rand((case["T"], case["N"]), generator=g, device="cuda") < 0.6).to(torch.uint8)
    return x, f, [1.0 / case["C"]] * case["C"], [int(c == 4) for c in range(case["C"])]


def _options(case):
    crit = CRIT5 if case["crit"] == 5 else CRIT4
    return dict(method=dc.DC_AHP if case["method"] == "ahp" else dc.DC_TOPSIS, crit=crit,
                cost=[int(c == dc.DC_CRIT_HOPS) for c in crit], routing=case["routing"])


def prepare(case, seed):
    if case["kind"] == "tiles":
        return dict(case=case, tiles=_matrices(case, seed))
    insts, reqs = _inputs(case, seed)
    if case["kind"] == "serving":
        return dict(case=case, insts=insts, reqs=reqs[0])
    s = dc.Scheduler(insts, mode=dc.DC_MODE_BATCHED if case["kind"] == "batched" else dc.DC_MODE_PLAIN,
                     **_options(case))
    buf = np.zeros(sum(map(len, reqs)), dc.RESULT_DTYPE)
    if case["kind"] == "online":
        return dict(case=case, s=s, reqs=reqs[0], buf=buf)
    for i, queue in enumerate(reqs):
        for q in queue:
            s.submit(q, instance=i)
    s.rewind()                          # uploads the queues
    return dict(case=case, s=s, buf=buf)


# ---------------------------------------------------------------- passes

def _decisions(res, **more):
    return dict({f: np.ascontiguousarray(res[f]) for f in ("status", "n", "failed_at", "host", "score")}, **more)


def run(state):
    return _PASS[state["case"]["kind"]](state)


def _online(state):
    s, buf = state["s"], state["buf"]
    ids = [s.submit(q) for q in state["reqs"]]
    res = s.schedule_array(buf)
    after = s.state(0)
    for rid, ok in zip(ids, res["status"].tolist()):
        if ok:
            s.release(rid)
    return _decisions(res, state=after)


def _replay(state):
    s = state["s"]
    s.rewind()
    return _decisions(s.schedule_array(state["buf"]), state=s.state(0))


def _batched(state):
    # the data centers' own states stay where they are, on the device: 256
    # read-backs are no part of a planning run
    state["s"].rewind()
    return _decisions(state["s"].schedule_array(state["buf"]))


def _serving(state):
    """Requests go in as fast as they are admitted, at most 64 undecided at
    a time; an accepted one departs once half the stream has followed it."""
    reqs, total = state["reqs"], len(state["reqs"])
    res, buf = np.zeros(total, dc.RESULT_DTYPE), np.zeros(256, dc.RESULT_DTYPE)
    with dc.Scheduler(state["insts"], mode=dc.DC_MODE_SERVING, **_options(state["case"])) as s:
        ids, done, gone = [], 0, 0
        while done < total:
            # departure r comes before request r + total // 2, so the order
            # of the commands, and with it every result, is fixed
            while len(ids) < total and len(ids) - done < 64:
                r = len(ids) - total // 2
                if gone <= r:
                    if done <= r:
                        break
                    if res[r]["status"] == 1 and s.release(ids[r]) != dc.DC_OK:
                        break
                    gone += 1
                    continue
                rid = s.try_submit(reqs[len(ids)])
                if rid is None:
                    break
                ids.append(rid)
            got = s.schedule_array(buf)
            res[done:done + len(got)] = got
            done += len(got)
        while s.pending():
            pass
        return _decisions(res, state=s.state(0))


def _tiles(state):
    x, f, w, cost = state["tiles"]
    best, score, scores = dc.topsis_tiles(x, w, cost=cost, feasible=f, scores=state["case"]["scores"])
    return dict(best=best, score=score, scores=scores) if scores is not None else dict(best=best, score=score)


_PASS = dict(online=_online, replay=_replay, batched=_batched, serving=_serving, tiles=_tiles)


def work(case):
    """Bytes: each input and output once.  Operations: per container step and
    server, the criteria (four per placed peer, one per criterion), then
    TOPSIS statistics and distances (nine per criterion) or, under AHP, a
    sort and two weighted counts over 17 ratios per criterion; as if every
    request were accepted."""
    if case["kind"] == "tiles":
        T, C, N = case["T"], case["C"], case["N"]
        return {"bytes": T * (4 * C * N + (N if case["feasible"] else 0) + (4 * N if case["scores"] else 0) + 8),
                "flops": T * N * (9 * C + 4)}
    N, C, n = case["k"] ** 3 // 4, case["crit"], (case["n_lo"] + case["n_hi"]) / 2
    R = case["requests"] if "requests" in case else case["instances"] * (case["r_lo"] + case["r_hi"]) / 2
    steps, pairs = R * n, R * max(n - 1, n * (n - 1) / 4)
    per = C * (math.log2(N) + 72) if case["method"] == "ahp" else 9 * C + 4
    return {"bytes": int(case.get("instances", 1) * 24 * N * 2 + steps * 24 + pairs * 16),
            "flops": int(N * (steps * (C + per) + 4 * pairs))}


# ---------------------------------------------------------------- 64 bits

def exact(case, seed):
    """The scores, in 64 bits.  Decisions are whole numbers.  A queue of many
    requests has no such value: where two servers' scores are closer than 32
    bits tell apart, either may be taken, and all that follows depends on it."""
    if case["kind"] == "tiles":
        return _exact_tiles(case, seed)
    if case["kind"] != "online" or case["requests"] > 64 or case["routing"]:
        return None
    insts, reqs = _inputs(case, seed)
    score = np.zeros((len(reqs[0]), dc.DC_MAX_CONTAINERS))
    site = _Site(insts[0], case)
    for r, q in enumerate(reqs[0]):
        score[r, :len(q.cpu)] = site.place(q)
    return dict(status=None, n=None, failed_at=None, host=None, score=score, state=None)


def _exact_tiles(case, seed):
    x, f, w, cost = _matrices(case, seed)
    score, scores = [], []
    w = torch.tensor(w, dtype=torch.float32, device=x.device).double()[None, :, None]
    flip = torch.tensor(cost, device=x.device).bool()[None, :, None]
    chunk = max(1, (1 << 24) // (case["C"] * case["N"]))
    for at in range(0, case["T"], chunk):
        v = x[at:at + chunk].double()
        norm = v.square().sum(2, keepdim=True).sqrt()
        v = torch.where(norm > 0, v / norm, torch.zeros_like(v)) * w
        hi, lo = v.amax(2, keepdim=True), v.amin(2, keepdim=True)
        up = (v - torch.where(flip, lo, hi)).square().sum(1).sqrt()
        dn = (v - torch.where(flip, hi, lo)).square().sum(1).sqrt()
        s = torch.where(up + dn > 0, dn / (up + dn), torch.zeros_like(up))
        if case["scores"]:
            scores.append(s)
        if f is not None:
            s = torch.where(f[at:at + chunk] != 0, s, torch.full_like(s, -1.0))
        score.append(s.amax(1).clamp(min=0.0))
    out = dict(best=None, score=torch.cat(score))
    return dict(out, scores=torch.cat(scores)) if case["scores"] else out


class _Site:
    """One data center and the placement of its requests, in 64 bits: every
    server scored from the definitions of sections V-B and V-C, the best on
    which the unit and its widest shortest paths fit taken."""

    def __init__(self, inst, case):
        self.k, self.h, self.N, self.case = inst.k, inst.k // 2, inst.k ** 3 // 4, case
        full = [inst.host_cpu, inst.host_ram, inst.bw_host_edge, inst.bw_edge_agg, inst.bw_agg_core]
        used = [0] * 5 if inst.host_used is None else [*inst.host_used, *inst.link_used]
        self.cpu, self.ram, self.up, ea, ac = (np.full(self.N, c, np.int64) - u for c, u in zip(full, used))
        self.ea, self.ac = ea.reshape(self.k, self.h, self.h), ac.reshape(self.k, self.h, self.h)   # [pod][edge|agg][...]
        self.placed = np.zeros(self.N, np.int64)
        u = np.arange(self.N)
        self.pod, self.edge = u // self.h ** 2, u // self.h % self.h

    def widest(self, v):
        """Bottleneck of the widest shortest path from every server to v."""
        pv, ev = self.pod[v], self.edge[v]
        core = np.minimum(self.ac, self.ac[pv][None]).max(2)                        # [pod][agg]
        core[pv] = 1 << 40
        tab = np.minimum(np.minimum(self.ea, self.ea[pv, ev]), core[:, None, :]).max(2)
        tab[pv, ev] = 1 << 40
        return np.minimum(np.minimum(self.up, self.up[v]), tab[self.pod, self.edge])

    def hops(self, v):
        same = self.pod == self.pod[v]
        h = np.where(same, np.where(self.edge == self.edge[v], 2, 4), 6)
        h[v] = 0
        return h

    def route(self, u, v):
        """Links (array, index) of the widest shortest path, lowest on ties."""
        pu, pv, eu, ev = self.pod[u], self.pod[v], self.edge[u], self.edge[v]
        links = [(self.up, u), (self.up, v)]
        if (pu, eu) != (pv, ev):
            b = np.minimum(np.minimum(self.ea[pu, eu], self.ea[pv, ev]), min(self.up[u], self.up[v]))
            if pu == pv:
                a = int(b.argmax())
            else:
                a, j = np.unravel_index(np.minimum(np.minimum(self.ac[pu], self.ac[pv]), b[:, None]).argmax(),
                                        (self.h, self.h))
                links += [(self.ac, (pu, a, j)), (self.ac, (pv, a, j))]
            links += [(self.ea, (pu, eu, a)), (self.ea, (pv, ev, a))]
        return links

    def commit(self, u, unit, peers):
        """Takes the unit's demand and its routes at server u, or nothing."""
        taken, routes = [], []
        for v, lo, hi in peers:
            if v == u:
                continue
            links = self.route(u, v)
            if min(a[i] for a, i in links) < lo:
                for a, i, b in taken:
                    a[i] += b
                return None
            for a, i in links:
                a[i] -= lo
                taken.append((a, i, lo))
            routes.append((links, hi - lo))
        for links, room in routes:
            add = min(room, min(a[i] for a, i in links))
            for a, i in links:
                a[i] -= add
                taken.append((a, i, add))
        for a, lo, hi in ((self.cpu, unit[0], unit[1]), (self.ram, unit[2], unit[3])):
            b = max(lo, min(hi, a[u]))
            a[u] -= b
            taken.append((a, u, b))
        self.placed[u] += 1
        taken.append((self.placed, u, -1))
        return taken

    def scores(self, cols, cost):
        X = np.stack(cols).astype(np.float64)
        w = float(np.float32(1.0 / len(cols)))
        if self.case["method"] == "topsis":
            norm = np.sqrt((X * X).sum(1, keepdims=True))
            V = np.divide(X, norm, out=np.zeros_like(X), where=norm > 0) * w
            hi, lo = V.max(1, keepdims=True), V.min(1, keepdims=True)
            flip = np.array(cost, bool)[:, None]
            up = np.sqrt(((V - np.where(flip, lo, hi)) ** 2).sum(0))
            dn = np.sqrt(((V - np.where(flip, hi, lo)) ** 2).sum(0))
            return np.divide(dn, up + dn, out=np.zeros_like(dn), where=up + dn > 0)
        total = np.zeros(self.N)
        for x, c in zip(cols, cost):
            val, back, cnt = np.unique(x, return_inverse=True, return_counts=True)
            hi, lo = np.maximum(val[:, None], val[None]), np.minimum(val[:, None], val[None])
            s = np.where(lo > 0, np.minimum(9, (2 * hi + lo) // np.maximum(2 * lo, 1)), 9)
            s = np.where(hi == lo, 1, s).astype(np.float64)
            larger = val[:, None] >= val[None] if not c else val[:, None] <= val[None]
            M = np.where(larger, s, 1.0 / s)                     # row value against column value
            col = (M * cnt[:, None]).sum(0)
            total += w * ((M / col * cnt).sum(1) / self.N)[back]
        return total

    def place(self, q):
        """Places the request; the score of each container's server (0 from
        the first pod without a server on).  All or nothing."""
        n = len(q.cpu)
        unit_of, first, seen = [], [], {}
        for i in range(n):
            key = i if q.pod is None or q.pod[i] < 0 else -1 - int(q.pod[i])
            if key not in seen:
                seen[key] = len(first)
                first.append(i)
            unit_of.append(seen[key])
        U = len(first)
        mx = [x if m is None else m for x, m in ((q.cpu, q.cpu_max), (q.ram, q.ram_max), (q.edges[:, 2], q.bw_max))]
        ask, lo, hi = np.zeros((U, 4), np.int64), np.zeros((U, U), np.int64), np.zeros((U, U), np.int64)
        for i, g in enumerate(unit_of):
            ask[g] += (q.cpu[i], mx[0][i], q.ram[i], mx[1][i])
        for (i, j, b), bx in zip(q.edges.tolist(), mx[2].tolist()):
            g, h = unit_of[i], unit_of[j]
            lo[g, h] += b
            lo[h, g] += b
            hi[g, h] += bx
            hi[h, g] += bx
        host, got, taken = [], np.zeros(U), []
        for g in range(U):
            peers = [(host[p], lo[g, p], hi[g, p]) for p in range(g) if lo[g, p] > 0]
            fits = (self.cpu >= ask[g, 0]) & (self.ram >= ask[g, 2])
            path, out, hop = self.up.copy(), np.zeros(self.N, np.int64), np.zeros(self.N, np.int64)
            for v, b, _ in peers:
                wide, away = self.widest(v), np.arange(self.N) != v
                fits &= ~away | (wide >= b)
                path = np.where(away, np.minimum(path, wide), path)
                out += away * b
                hop += self.hops(v)
            fits &= self.up >= out
            if self.case["crit"] == 5:
                cols, cost = [self.cpu, self.ram, self.up, path, hop], [0, 0, 0, 0, 1]
            else:
                cols, cost = [self.cpu, self.ram, self.placed > 0, path], [0] * 4
            s = self.scores([np.asarray(c, np.int64) for c in cols], cost)
            mine = None
            for u in np.lexsort((np.arange(self.N), -s)):
                if fits[u]:
                    mine = self.commit(u, ask[g], peers)
                    if mine is not None:
                        break
            if mine is None:
                for a, i, b in reversed(taken):
                    a[i] += b
                break
            taken += mine
            host.append(int(u))
            got[g] = s[u]
        return got[unit_of]
