// Cooperative container step for large data centers: one workgroup per pod
// (k workgroups, launched cooperatively so that all are resident).  Each
// workgroup builds the path tables for its own pod's aggregation and edge
// switches, scores its pod's servers; the column statistics and the
// capacity sums are exchanged through tagged per-workgroup records, the
// argmax and the commit's outcome through tagged slots (selection rounds),
// so that a step has no grid barrier; workgroup 0 commits.  Same arithmetic as the single-workgroup step, so
// results are bit-identical.  Used by the plain form (one cooperative launch
// per container step) and the serving form (one persistent cooperative
// kernel) when k is large.
#pragma once
#include "dc_serve.hpp"

namespace dcs {

// Threads per pod workgroup.  The step is bound by memory latency and the
// waits between workgroups: a session of 300 requests at k = 48 (576 servers a
// pod) took 62.6 ms with 256 threads, 60.3 with 512, 65.8 with 576 and 84.7
// with 1,024, where registers spill.  In smaller pods the fewer waves of 256
// threads meet sooner: a queue of 100 requests took 14.3 ms with 256 and 15.0
// with 512 at k = 22 (121 servers a pod), 15.1 and 15.8 at k = 32, 17.6 and
// 17.7 at k = 40, 17.7 and 17.3 at k = 48, 22.2 and 21.1 at k = 56.  One size
// serves them all so far.
constexpr int kGridBlock = 512;

// Cross-workgroup state, in device memory.
struct GridCtl {
    unsigned *count, *gen;        // grid barrier: arrivals, generation
    int *err;                     // set when a barrier wait timed out
    unsigned long long *kslot;    // [2][G] per-workgroup best key of a selection round, tagged
    unsigned long long *rflag;    // outcome of a selection round's commit, tagged
    unsigned long long *rec;      // [kRecWords][pods] per-workgroup records of a step, tagged (below)
    int pods;                     // workgroups that own a pod (the first k)
    int wgs;                      // workgroups that take part in the rounds and barriers (the first)
    unsigned *round;              // selection rounds so far (kept across launches)
    unsigned *join;               // [2] entry of the queue kernels: arrivals, decision
    // serving form: commands as the fetching workgroup hands them out, and
    // their way back (below)
    unsigned long long *cmd;      // [kCmdRing][kCmdWords], tagged with position + 1
    long long *times;             // [kCmdRing][2] device clock when the command was seen, and at its decision
    int *done, *reported;         // commands completed / reported to the host
};

// Selection rounds.  Round r of the argmax and commit needs no grid barrier:
// each workgroup publishes its best key in its own slot of set r & 1 as one
// 64-bit word, tagged with r, which a wave of every workgroup polls until all
// slots carry r (the payload is the word itself, so no fence is needed);
// workgroup 0 then commits and publishes the outcome tagged with r (release),
// which the others poll for (acquire).  A round that ends with no server left
// has no outcome, so the outcome's word may be any number of rounds old: it
// carries 31 bits of r (rec_tag below), where the slots, written in every
// round, need only tell r from r - 2.  A workgroup publishes round r + 2 in
// the same slot only after the outcome of round r + 1, which workgroup 0
// gives only after reading every slot of round r + 1, so nothing is
// overwritten before every workgroup has read it.  Keys are packed as
// (score bits + 1) << 17 | (2^17 - 1 - server) (servers below 2^17), the tag
// in bits 47..63; tags never are 0, which the slots hold initially.
constexpr int kRoundTagShift = 47;
constexpr unsigned long long kRoundPayload = (1ull << kRoundTagShift) - 1;
__device__ __forceinline__ unsigned long long round_tag(unsigned r) {
    return static_cast<unsigned long long>((r & 0xffffu) | 0x10000u) << kRoundTagShift;
}
__device__ __forceinline__ unsigned long long round_key(unsigned long long kb) {
    if (!kb) return 0ull;
    const unsigned u = ~static_cast<unsigned>(kb);
    return ((kb >> 32) << 17) | (0x1ffffu - u);
}

// Wave: waits until the G slots of round r all carry its tag and returns the
// largest payload, or sets bad when the wait timed out or a workgroup
// reported an error.
__device__ __forceinline__ unsigned long long round_max(const GridCtl &g, unsigned r, long long timeout,
                                                        bool &bad) {
    const int lane = threadIdx.x & (kWave - 1), G = g.wgs;
    const unsigned long long *sl = g.kslot + (r & 1) * G, tag = round_tag(r);
    const long long t0 = dev_clock();
    for (;;) {
        bool ok = true;
        unsigned long long m = 0;
        for (int x = lane; x < G; x += kWave) {
            const unsigned long long v = __hip_atomic_load(sl + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok &= (v & ~kRoundPayload) == tag;
            const unsigned long long pv = v & kRoundPayload;
            m = pv > m ? pv : m;
        }
        if (__all(ok)) {
            const unsigned hiw = wave_umax(static_cast<unsigned>(m >> 32));
            const unsigned low = wave_umax(static_cast<unsigned>(m >> 32) == hiw ? static_cast<unsigned>(m) : 0u);
            return (static_cast<unsigned long long>(hiw) << 32) | low;
        }
        if (__hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || dev_clock() - t0 > timeout) {
            if (lane == 0) __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bad = true;
            return 0ull;
        }
    }
}

// Tag of a word in its high half: 31 bits of a round's number, the top bit
// set.
__device__ __forceinline__ unsigned long long rec_tag(unsigned r) {
    return static_cast<unsigned long long>(r | 0x80000000u) << 32;
}
__device__ __forceinline__ bool rec_has(unsigned long long v, unsigned long long tag) { return (v >> 32) == (tag >> 32); }

// Thread: waits for workgroup 0's outcome of round r; -1 when the wait
// timed out or a workgroup reported an error.
__device__ __forceinline__ int round_outcome(const GridCtl &g, unsigned r, long long timeout) {
    const unsigned long long tag = rec_tag(r);
    const long long t0 = dev_clock();
    for (;;) {
        const unsigned long long v = __hip_atomic_load(g.rflag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (rec_has(v, tag)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            return static_cast<int>(v & 3u);
        }
        if (__hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || dev_clock() - t0 > timeout) {
            __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Grid barrier over the first g.wgs workgroups, all co-resident, with agent-scope
// release / acquire.  A wait longer than `timeout` device ticks sets *err;
// every barrier returns false once *err is set, so all workgroups leave.
// Ordering: each arrival's fetch_add releases the workgroup's writes (after
// the block barrier) and acquires the earlier arrivals'; the last arrival
// publishes the next generation with a release store; the others poll it
// with relaxed loads and take one acquire fence once it has changed.  The
// generation is read before arriving, which the release of the fetch_add
// keeps in place.  No other fence is needed, and on a device of several
// XCDs each one costs a second-level cache writeback or invalidation.
__device__ __forceinline__ bool grid_sync(const GridCtl &g, int *lds_flag, long long timeout) {
    __syncthreads();
    if (threadIdx.x == 0) {
        int bad = __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!bad) {
            const unsigned gen = __hip_atomic_load(g.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned arrived = __hip_atomic_fetch_add(g.count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (arrived == static_cast<unsigned>(g.wgs) - 1) {
                __hip_atomic_store(g.count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(g.gen, gen + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const long long t0 = dev_clock();
                while (__hip_atomic_load(g.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gen) {
                    if (__hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) { bad = 1; break; }
                    if (dev_clock() - t0 > timeout) {
                        __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        bad = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
        }
        *lds_flag = bad;
    }
    __syncthreads();
    return !*lds_flag;
}

// Records of a step: instead of a grid barrier, each workgroup publishes
// its column-statistics partials, its edge switches' and its pod's summed
// residuals (and workgroup 0 the trace slot) as 64-bit words, the value in
// the low half and in the high half rec_tag of the step's
// first selection round (never 0, which the words hold
// initially); a reader polls a word until it carries that tag, so no fence
// is needed.  Every word is written at every step, a step has fewer than
// 2^31 rounds, so a word read with the current tag was written in this step.
// A workgroup writes the next step's record only after this step's last
// selection round, whose outcome needs every workgroup's key, which each
// publishes after it has read the records.  A wave reads one word of every
// workgroup at once, so the words are laid out by word, then workgroup: one
// poll then takes a few cache lines a word instead of one per workgroup.
constexpr int kRecWords = 80;
constexpr int kRecCapE = 5 * kMaxCrit;            // then h edge switches (h <= 32)
constexpr int kRecCapP = kRecCapE + 32;
constexpr int kRecTrace = kRecCapP + 1;
static_assert(kRecTrace < kRecWords, "record layout");

__device__ __forceinline__ void rec_put(const GridCtl &g, int w, int x, unsigned long long tag, int v) {
    __hip_atomic_store(g.rec + x * g.pods + w, tag | static_cast<unsigned>(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long rec_load(const GridCtl &g, int w, int x) {
    return __hip_atomic_load(g.rec + x * g.pods + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread: n words of the records (workgroup ws[j], word xs[j]) once all
// carry tag, every poll with all its loads in flight together; false when
// the wait timed out or a workgroup reported an error.
template <int NW>
__device__ __forceinline__ bool rec_get(const GridCtl &g, int n, const int (&ws)[NW], const int (&xs)[NW],
                                        unsigned long long tag, long long timeout, int (&v)[NW]) {
    const long long t0 = dev_clock();
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int j = 0; j < NW; ++j)
            if (j < n) {
                const unsigned long long r = rec_load(g, ws[j], xs[j]);
                ok &= rec_has(r, tag);
                v[j] = static_cast<int>(static_cast<unsigned>(r));
            }
        if (ok) return true;
        if (__hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || dev_clock() - t0 > timeout) {
            __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// LDS of the cooperative step (per workgroup): peers, the own pod's state,
// tables and capacities, per-server scratch of the pod, statistics slots.
struct GSmem {
    int4 *pk;                     // [kMaxN] packed peers (as in Smem)
    int *wst;                     // [kStatFields][kMaxWaves]
    int *misc;                    // [M_MISC]
    int *own;                     // [6][hh] the own pod's residuals, as in State
    int *capE;                    // [h] own edge switches, summed
    int *tabT, *tabE, *peerE;     // [kMaxN][h] path tables; the peers' edge-aggregation residuals
    int *xs;                      // [nc+6][hh]
};

// Residuals of the own pod kept in LDS, and the tables of a step.
__host__ __device__ inline size_t own_ints(int h, int hh) { return align4(6 * (size_t)hh) + align4(h); }
__host__ __device__ inline size_t tab_ints(int h) { return 3 * align4((size_t)kMaxN * h); }
__device__ inline int *carve_tabs(GSmem &s, int *p, int h) {
    s.tabT = p; p += align4((size_t)kMaxN * h);
    s.tabE = p; p += align4((size_t)kMaxN * h);
    s.peerE = p; p += align4((size_t)kMaxN * h);
    return p;
}

__host__ __device__ inline size_t gsmem_bytes(int h, int hh, int nc) {
    return sizeof(int4) * kMaxN +
           sizeof(int) * (kStatFields * kMaxWaves + M_MISC + own_ints(h, hh) + tab_ints(h) + (size_t)(nc + 6) * hh);
}

__device__ inline GSmem gcarve(char *base, int h, int hh, int nc) {
    GSmem s;
    s.pk = reinterpret_cast<int4 *>(base);
    int *p = reinterpret_cast<int *>(base + sizeof(int4) * kMaxN);
    s.wst = p; p += kStatFields * kMaxWaves;
    s.misc = p; p += M_MISC;
    s.own = p; p += align4(6 * (size_t)hh);
    s.capE = p; p += align4(h);
    s.xs = carve_tabs(s, p, h);
    return s;
}

// max_j min(x[j], y[j]) over n entries (n % 4 == 0: 16-byte aligned rows)
template <class X, class Y>
__device__ __forceinline__ int max_min(X x, Y y, int n) {
    int val = 0;
    if ((n & 3) == 0) {
#pragma unroll 4
        for (int j = 0; j < n; j += 4) {
            const int4 a = *reinterpret_cast<const int4 *>(x + j), b = *reinterpret_cast<const int4 *>(y + j);
            val = max(val, max(max(min(a.x, b.x), min(a.y, b.y)), max(min(a.z, b.z), min(a.w, b.w))));
        }
    } else {
#pragma unroll 8
        for (int j = 0; j < n; ++j) val = max(val, min(x[j], y[j]));
    }
    return val;
}

// Peers, own capacities, path tables and criteria of a container step, for
// the servers of this workgroup's pod (w = blockIdx.x < k).  emit(x, f, get)
// receives server x of the pod, its feasibility and its criteria get(c), in
// one thread per server.  The deficit slots and M_OK are reset here, before
// the first barrier.  The pod's residuals stay in LDS from step to step and
// are read again only where a commit may have changed them (`stale`), so a
// step waits for memory once, for the peers' residuals, instead of once per
// stage: see grid_select for who sets stale.  misc[M_CAPP] keeps the pod's
// summed aggregation-core residual.
template <int BS, int CS, class Emit>
__device__ __forceinline__ void grid_criteria(const Topo &t, const State &st, const Method &m, const GSmem &sm,
                                              const StepIn &s, const ReqView &rv, bool stale, Emit emit) {
    const int w = blockIdx.x, h = t.h, hh = t.hh, P = s.P, ubase = w * hh;
    int *own_up = sm.own + 3 * hh, *own_ea = sm.own + 4 * hh, *own_ac = sm.own + 5 * hh;
    // ---- A: everything a step reads from memory.  Peers, their edge
    // switches' rows, table T (against the peers' aggregation-core rows)
    for (int p = threadIdx.x; p < P; p += BS) {
        const int v = rv.hosts[rv.pj[p]];
        sm.pk[p] = make_int4(v, edge_of(t, v) | (pod_of(t, v) << 16), rv.pbw[p], st.up[v]);
    }
    if (threadIdx.x < 6) sm.misc[M_DH0 + threadIdx.x] = (threadIdx.x & 1) ? -1 : kBig;
    if (threadIdx.x == 6) sm.misc[M_OK] = 0;
    if (stale) {
        // the six arrays are contiguous, N entries each
        const int n = 6 * hh;
        if ((hh & 3) == 0) {
            for (int x = 4 * threadIdx.x; x < n; x += 4 * BS) {
                const int f = x / hh;
                *reinterpret_cast<int4 *>(sm.own + x) =
                    *reinterpret_cast<const int4 *>(st.cpu + (size_t)f * t.N + ubase + (x - f * hh));
            }
        } else {
            for (int x = threadIdx.x; x < n; x += BS) {
                const int f = x / hh;
                sm.own[x] = st.cpu[(size_t)f * t.N + ubase + (x - f * hh)];
            }
        }
    }
    for (int it = threadIdx.x; it < P * h; it += BS) {
        const int pc = it / h, a = it - pc * h;
        const int v = rv.hosts[rv.pj[pc]], pv = pod_of(t, v);
        sm.peerE[it] = st.ea[edge_of(t, v) * h + a];
        const int *y = st.ac + (pv * h + a) * h;
        int val = 0;
        if (pv != w) val = stale ? max_min(st.ac + (w * h + a) * h, y, h) : max_min(own_ac + a * h, y, h);
        sm.tabT[it] = val;
    }
    __syncthreads();
    // ---- B: table E of the pod's edge switches, own capacities
    if (stale) {
        for (int e = BS - 1 - static_cast<int>(threadIdx.x); e < h; e += BS) {
            int se = 0;
            for (int a = 0; a < h; ++a) se += own_ea[e * h + a];
            sm.capE[e] = se;
        }
        if (threadIdx.x < kWave) {
            int cp = 0;
            for (int x = threadIdx.x; x < hh; x += kWave) cp += own_ac[x];
            cp = wave_sum(cp);
            if (threadIdx.x == 0) sm.misc[M_CAPP] = cp;
        }
    }
    for (int it = threadIdx.x; it < P * h; it += BS) {
        const int pc = it / h, e = it - pc * h;
        const int ed = sm.pk[pc].y, ev = ed & 0xffff, pv = ed >> 16, eg = w * h + e;
        int val = 0;
        if (eg != ev) {
            const int *x = own_ea + e * h, *y = sm.peerE + pc * h, *T = sm.tabT + pc * h;
            const int lim = pv != w ? 0 : kBig;
            for (int a = 0; a < h; ++a) val = max(val, min(min(x[a], y[a]), max(T[a], lim)));
        }
        sm.tabE[it] = val;
    }
    __syncthreads();
    // ---- C: criteria of the pod's servers
    const int capP_own = sm.misc[M_CAPP];
    for (int x = threadIdx.x; x < hh; x += BS) {
        const int u = ubase + x;
        const int up_u = own_up[x], el = edge_of(t, x), eu = w * h + el;
        const int cpu_u = sm.own[x], ram_u = sm.own[hh + x];
        int pbw_acc = up_u, up_acc = 0, hop_acc = 0, oute = 0, outp = 0;
        int feas = (cpu_u >= s.cpu) & (ram_u >= s.ram);
        for (int pc = 0; pc < P; ++pc) {
            const int4 pk = sm.pk[pc];
            const int v = pk.x, bw = pk.z, ev = pk.y & 0xffff, pv = pk.y >> 16;
            const bool rem = v != u, far = ev != eu;
            int wv = min(up_u, pk.w);
            wv = far ? min(wv, sm.tabE[pc * h + el]) : wv;
            pbw_acc = rem ? min(pbw_acc, wv) : pbw_acc;
            up_acc += rem ? bw : 0;
            hop_acc += !rem ? 0 : !far ? 2 : (pv == w ? 4 : 6);
            feas &= (!rem) | (wv >= bw);
            oute += (rem & far) ? bw : 0;
            outp += (rem & far & (pv != w)) ? bw : 0;
        }
        feas &= (up_u >= up_acc);
        if (P > 0 && !m.route_end) feas &= (sm.capE[el] >= oute) & (capP_own >= outp);
        emit(x, feas, [&](int c) -> int {
            switch (crit_at<CS>(m, c)) {
            case CRIT_CPU: return cpu_u;
            case CRIT_RAM: return ram_u;
            case CRIT_ACTIVE: return sm.own[2 * hh + x] > 0 ? 1 : 0;
            case CRIT_PATHBW: return pbw_acc;
            case CRIT_UPLINK: return up_u;
            default: return hop_acc;
            }
        });
    }
}

// Peer-side deficits (server uplink, edge switch, pod) as in the
// single-workgroup step, by thread p for peer p (me its packed record, capE
// and capP its edge switch's and pod's summed residuals); they only narrow
// the candidates.  The slots were reset by grid_criteria.
__device__ __forceinline__ void grid_deficits(const GSmem &sm, int P, const int4 &me, int capE, int capP) {
    const int v = me.x, e = me.y & 0xffff, d = me.y >> 16;
    int sh = 0, se = 0, sp = 0;
    for (int q = 0; q < P; ++q) {
        const int4 o = sm.pk[q];
        sh += o.x == v ? o.z : 0;
        se += (o.y & 0xffff) == e ? o.z : 0;
        sp += (o.y >> 16) == d ? o.z : 0;
    }
    if (me.w < sh) { atomicMin(sm.misc + M_DH0, v); atomicMax(sm.misc + M_DH1, v); }
    if (capE < se) {
        atomicMin(sm.misc + M_DE0, e);
        atomicMax(sm.misc + M_DE1, e);
    }
    if (capP < sp) {
        atomicMin(sm.misc + M_DP0, d);
        atomicMax(sm.misc + M_DP1, d);
    }
}

// Whether the deficits leave server x of pod w a candidate.
struct Deficits {
    int dh0, dh1, de0, de1, dp0, dp1;
};
__device__ __forceinline__ Deficits read_deficits(const GSmem &sm) {
    return Deficits{sm.misc[M_DH0], sm.misc[M_DH1], sm.misc[M_DE0], sm.misc[M_DE1], sm.misc[M_DP0], sm.misc[M_DP1]};
}
__device__ __forceinline__ bool deficits_allow(const Topo &t, const Deficits &d, int w, int x) {
    int f = (d.dh1 < 0) | ((d.dh0 == d.dh1) & (w * t.hh + x == d.dh0));
    f &= (d.de1 < 0) | ((d.de0 == d.de1) & (w * t.h + edge_of(t, x) == d.de0));
    f &= (d.dp1 < 0) | ((d.dp0 == d.dp1) & (w == d.dp0));
    return f;
}

// Selection rounds of a step (global argmax, commit by workgroup 0,
// retries).  key_of(x): the score key of the pod's server x, 0 when it is
// no candidate (feas[x] == 0 masks it); a workgroup without a pod (nx = 0)
// only follows.  Returns false when the request was rejected at this
// container, or a wait failed.  stale: whether this pod's residuals may have
// changed.  A commit changes those of the chosen server's pod and of the
// peers' pods, a rollback or the routing at a request's end any.
// TOGETHER: see commit_wave.
template <int BS, bool TOGETHER, class KeyFn>
__device__ __forceinline__ bool grid_select(const Topo &t, const State &st, const Method &m, const Batch &b,
                                            const GSmem &sm, const GridCtl &g, long long timeout, const StepIn &s,
                                            const ReqView &rv, unsigned &rnd, bool &stale, int nx, int *feas, KeyFn key_of) {
    const int w = blockIdx.x, G = g.wgs, ubase = w * t.hh, P = s.P;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    // the workgroup's best key (largest packed key) into LDS slot 0..1
    auto wg_best = [&]() {
        unsigned long long kb = 0;
        for (int x = threadIdx.x; x < nx; x += BS) {
            const unsigned long long k = key_of(x);
            kb = k > kb ? k : kb;
        }
        unsigned hiw = wave_umax(static_cast<unsigned>(kb >> 32));
        unsigned low = wave_umax(static_cast<unsigned>(kb >> 32) == hiw ? static_cast<unsigned>(kb) : 0u);
        if (lane == 0) {
            sm.wst[wid] = static_cast<int>(hiw);
            sm.wst[kMaxWaves + wid] = static_cast<int>(low);
        }
        __syncthreads();
        if (threadIdx.x < kWave) {
            const unsigned hi = lane < BS / kWave ? static_cast<unsigned>(sm.wst[lane]) : 0u;
            const unsigned lo = lane < BS / kWave ? static_cast<unsigned>(sm.wst[kMaxWaves + lane]) : 0u;
            hiw = wave_umax(hi);
            low = wave_umax(hi == hiw ? lo : 0u);
            if (lane == 0)
                *reinterpret_cast<unsigned long long *>(sm.misc + M_KEY) =
                    round_key((static_cast<unsigned long long>(hiw) << 32) | low);
        }
    };
    wg_best();
    stale = true;                              // until the container is placed
    for (;;) {
        const unsigned r = rnd++;
        if (threadIdx.x == 0)
            __hip_atomic_store(g.kslot + (r & 1) * G + w,
                               round_tag(r) | *reinterpret_cast<const unsigned long long *>(sm.misc + M_KEY),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (threadIdx.x < kWave) {
            bool bad = false;
            const unsigned long long kb = round_max(g, r, timeout, bad);
            if (lane == 0) {
                *reinterpret_cast<unsigned long long *>(sm.wst + 2 * kMaxWaves) = kb;
                sm.misc[M_OK] = bad;
            }
        }
        __syncthreads();
        if (sm.misc[M_OK]) return false;
        const unsigned long long kb = *reinterpret_cast<const unsigned long long *>(sm.wst + 2 * kMaxWaves);
        if (kb == 0) {                                                        // no server left
            if (w == 0) rollback_request<BS>(t, st, b, s.r, s.i);
            grid_sync(g, sm.misc + M_OK, timeout);
            return false;
        }
        const int u = static_cast<int>(0x1ffffu - static_cast<unsigned>(kb & 0x1ffffu));
        if (w == 0) {
            // workgroup 0 commits: 1 placed, 0 retry with the next server,
            // 2 request rejected when its links were routed at its end
            if (threadIdx.x < kWave) {
                // commit_wave reads the peer servers from LDS; its routing
                // uses the global state
                Smem cs;
                cs.pk = sm.pk;
                const bool ok = commit_wave<TOGETHER>(t, st, b, u, s, m.route_end ? 0 : P, cs, b.pbmax + s.p0, lane);
                if (lane == 0) {
                    sm.misc[M_ROUTE + 1] = ok;
                    if (ok) {
                        b.host[s.g] = u;
                        b.score[s.g] = __uint_as_float(static_cast<unsigned>(kb >> 17) - 1u);
                        if (s.i == s.n - 1) b.tse[s.r] = dev_clock();
                    }
                }
            }
            __syncthreads();
            int res = sm.misc[M_ROUTE + 1];
            if (res && m.route_end && s.i == s.n - 1)
                res = route_request_end<BS>(t, st, b, sm.misc + M_ROUTE, s, rv,
                                            [&](int q) { return q == s.i ? u : rv.hosts[q]; }) ? 1 : 2;
            __syncthreads();
            if (threadIdx.x == 0) {
                __hip_atomic_store(g.rflag, rec_tag(r) | static_cast<unsigned>(res), __ATOMIC_RELEASE,
                                   __HIP_MEMORY_SCOPE_AGENT);
                sm.misc[M_RES] = res;
            }
        } else if (threadIdx.x == 0) {
            sm.misc[M_RES] = round_outcome(g, r, timeout);
        }
        __syncthreads();
        const int ok = sm.misc[M_RES];
        if (ok < 0 || ok == 2) return false;
        if (ok) {
            if (rv.hosts_out && threadIdx.x == 0) rv.hosts_out[s.i] = u;
            stale = (m.route_end && s.i == s.n - 1) || pod_of(t, u) == w ||
                    __any(lane < P && (sm.pk[lane].y >> 16) == w);
            __syncthreads();
            return true;
        }
        if (u - ubase >= 0 && u - ubase < nx) {                               // owner masks it and rescans
            if (threadIdx.x == 0) feas[u - ubase] = 0;
            __syncthreads();
            wg_best();
        }
        __syncthreads();
    }
}

// One container step on the pod of this workgroup (w = blockIdx.x).
// rv.hosts_out, when given, is this workgroup's LDS copy of the request's
// servers.  Returns false when the request was rejected at this container.
template <int BS, int CS = 0>
__device__ __forceinline__ bool grid_topsis_step(const Topo &t, const State &st, const Method &m, const Batch &b,
                                                 const GSmem &sm, const GridCtl &g, long long timeout, const StepIn &s,
                                                 const ReqView &rv, const Trace &tr, unsigned &rnd, bool &stale) {
    const int w = blockIdx.x, G = g.wgs, h = t.h, hh = t.hh, nc = crit_count<CS>(m);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int P = s.P, ubase = w * hh;
    int *xs = sm.xs;
    const unsigned long long stag = rec_tag(rnd);     // this step's records
    int my_slot = -1;                                   // trace slot (workgroup 0, thread 0)
    if (w == 0 && threadIdx.x == 0) {
        if (s.i == 0) b.tsb[s.r] = dev_clock();
        if (tr.stride > 0) my_slot = trace_slot(tr, 0, b.rid[s.r], s.i);
    }
    // partial column statistics of the pod's servers
    unsigned long long s2[kMaxCrit];
    int mx[kMaxCrit], mn[kMaxCrit];
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) { s2[c] = 0; mx[c] = -kBig - 1; mn[c] = kBig; }
    grid_criteria<BS, CS>(t, st, m, sm, s, rv, stale, [&](int x, int f, auto get) {
        xs[nc * hh + x] = f;
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) {
            if (c >= nc) break;
            const int v = get(c);
            xs[c * hh + x] = v;
            s2[c] += static_cast<unsigned long long>(static_cast<long long>(v) * v);
            mx[c] = max(mx[c], v);
            mn[c] = min(mn[c], v);
        }
    });
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        if (c >= nc) break;
        const int c0 = wave_sum(static_cast<int>(s2[c] & 0x1ffffu));
        const int c1 = wave_sum(static_cast<int>((s2[c] >> 17) & 0x1ffffu));
        const int c2 = wave_sum(static_cast<int>(s2[c] >> 34));
        const int hi = wave_max(mx[c]), lo = wave_min(mn[c]);
        if (lane < 5) sm.wst[(5 * c + lane) * kMaxWaves + wid] =
            lane == 0 ? c0 : lane == 1 ? c1 : lane == 2 ? c2 : lane == 3 ? hi : -lo;
    }
    __syncthreads();
    // this workgroup's record: statistics partials, own capacities for the
    // other pods' checks, and (workgroup 0) the trace slot
    for (int f = threadIdx.x; f < 5 * nc; f += BS) {
        int v = (f % 5) < 3 ? 0 : -kBig - 1;
        for (int x = 0; x < BS / kWave; ++x) {
            const int pv = sm.wst[f * kMaxWaves + x];
            v = (f % 5) < 3 ? v + pv : max(v, pv);
        }
        rec_put(g, w, f, stag, v);
    }
    for (int e = threadIdx.x; e < h; e += BS) rec_put(g, w, kRecCapE + e, stag, sm.capE[e]);
    if (threadIdx.x == 0) {
        rec_put(g, w, kRecCapP, stag, sm.misc[M_CAPP]);
        if (w == 0) rec_put(g, 0, kRecTrace, stag, my_slot);
    }
    // ---- D: block totals, peer-side deficits, scores, workgroup best
    // One poll for all a wave needs from the records, until every word
    // carries this step's tag: wave 0 takes the statistics, lane x those of
    // workgroup x (G <= 64; the lanes past G read workgroup 0's and count
    // identities instead), wave 1 the capacities of peer x's edge switch and
    // pod (P <= 63).  The other waves wait at the barrier: with every wave
    // polling, the polls of 48 workgroups held one another up (a step at
    // 1,024 threads took 1.4 times as long as at 256).
    constexpr int NF = 5 * (CS ? CS : kMaxCrit);
    static_assert(BS >= 2 * kWave, "statistics and capacities are waited for by two waves");
    float *fac = reinterpret_cast<float *>(sm.wst) + 4 * kMaxWaves;
    bool bad = false;
    if (wid == 0) {
        int ww[NF], wx[NF], fv[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            ww[f] = lane < G ? lane : 0;
            wx[f] = f;
        }
        bad = !rec_get(g, 5 * nc, ww, wx, stag, timeout, fv);
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) {
            if (c >= nc || 5 * c >= NF) continue;
#pragma unroll
            for (int j = 0; j < 5; ++j) fv[5 * c + j] = lane < G ? fv[5 * c + j] : (j < 3 ? 0 : -kBig - 1);
            const int a0 = wave_sum(fv[5 * c]), a1 = wave_sum(fv[5 * c + 1]), a2 = wave_sum(fv[5 * c + 2]);
            const unsigned long long S2 = static_cast<unsigned long long>(static_cast<unsigned>(a0)) +
                                          (static_cast<unsigned long long>(static_cast<unsigned>(a1)) << 17) +
                                          (static_cast<unsigned long long>(static_cast<unsigned>(a2)) << 34);
            const int hi = wave_max(fv[5 * c + 3]), lo = -wave_max(fv[5 * c + 4]);
            if (lane == 0) {
                fac[c] = S2 ? (m.w[c] * m.w[c]) / static_cast<float>(S2) : 0.0f;
                fac[kMaxCrit + c] = static_cast<float>(crit_cost<CS>(m, c) ? lo : hi);
                fac[2 * kMaxCrit + c] = static_cast<float>(crit_cost<CS>(m, c) ? hi : lo);
            }
        }
    } else if (wid == 1 && lane < P) {
        const int4 me = sm.pk[lane];
        const int e = me.y & 0xffff, d = me.y >> 16;
        const int ww[2] = {e / h, d}, wx[2] = {kRecCapE + e % h, kRecCapP};
        int cv[2];
        bad = !rec_get(g, 2, ww, wx, stag, timeout, cv);
        grid_deficits(sm, P, me, cv[0], cv[1]);
    }
    int slot = -1;
    if (tr.stride > 0) {
        const int zw[1] = {0}, zx[1] = {kRecTrace};
        int zv[1];
        bad |= !rec_get(g, 1, zw, zx, stag, timeout, zv);
        slot = zv[0];
    }
    if (bad) sm.misc[M_OK] = 1;
    __syncthreads();
    if (sm.misc[M_OK]) return false;
    const Deficits df = read_deficits(sm);
    float q[kMaxCrit], ap[kMaxCrit], am[kMaxCrit];
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        q[c] = ap[c] = am[c] = 0.f;
        if (c >= nc) continue;
        q[c] = fac[c];
        ap[c] = fac[kMaxCrit + c];
        am[c] = fac[2 * kMaxCrit + c];
    }
    auto key_of = [&](int x) -> unsigned long long {
        if (!xs[nc * hh + x] || !(m.route_end || deficits_allow(t, df, w, x))) return 0ull;
        return score_key(topsis_close(nc, [&](int c) { return xs[c * hh + x]; }, q, ap, am), ubase + x);
    };
    if (slot >= 0)
        for (int x = threadIdx.x; x < hh; x += BS)
            tr.scores[static_cast<size_t>(slot) * t.N + ubase + x] =
                topsis_close(nc, [&](int c) { return xs[c * hh + x]; }, q, ap, am);
    return grid_select<BS, CS != 0>(t, st, m, b, sm, g, timeout, s, rv, rnd, stale, hh, xs + nc * hh, key_of);
}

}  // namespace dcs

namespace dcs {

// LDS of the request prefetch after the cooperative step's region.
__device__ __forceinline__ int *grid_req_lds(char *dsm, int h, int hh, int nc) {
    return reinterpret_cast<int *>(dsm + align4(gsmem_bytes(h, hh, nc) / sizeof(int)) * sizeof(int));
}

// Plain form, large data centers: one cooperative launch per container step.
// K > 0: k = K fat-trees on the four default criteria, as compile-time
// constants (as in the resident kernel); K = 0: any k, on those criteria
// (CS = 4) or any (CS = 0).
template <int BS, int K, int CS>
__global__ __launch_bounds__(BS) void k_topsis_grid(Params p, GridCtl g, long long timeout) {
    extern __shared__ __align__(16) char dsm[];
    // every workgroup leaves before any wait: the request was rejected at an
    // earlier step, or a wait of an earlier launch timed out (the launches of
    // a batch's steps are queued together, and a step after a failed one
    // would read the missing peer's server as -1)
    if (p.b.status[p.s.r] == 0 || __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const Topo t = topo_of<K>(p.t);
    const GSmem sm = gcarve(dsm, t.h, t.hh, crit_count<CS>(p.m));
    unsigned rnd = __hip_atomic_load(g.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool stale = true;
    grid_topsis_step<BS, CS>(t, p.st, p.m, p.b, sm, g, timeout, p.s, plain_view(p), p.tr, rnd, stale);
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(g.round, rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- serving form
// Large data centers: the persistent loop of k_serve over one workgroup per
// pod, and two more that talk to the host.  Host memory is a microsecond or
// two away in each direction, and a command used to cross it four times with
// every workgroup waiting (poll, barrier, request, completion): 40 us of a
// request.  Now the fetching workgroup polls the command ring, copies each
// request into its device slot and hands the command out as tagged words, up
// to kCmdAhead commands before they are reported; the reporting workgroup
// turns finished commands into completion records.  The pods only wait for
// device memory.  A session of 300 requests at k = 48: 57.1 -> 53.1 ms.
//
// Waits: the fetcher leaves after idle_ticks with nothing to do, handing out
// a stop; pods and reporter leave at that stop; every wait also ends when
// g.err is set, and the pods' wait for a command is bounded.
constexpr int kCmdRing = 8, kCmdAhead = 4, kCmdWords = 6;
static_assert(kCmdAhead < kCmdRing, "an entry is written again only after its command was reported");
enum { CW_TYPE = 0, CW_N, CW_NPAIR, CW_SLOT, CW_RID, CW_GOT };

__device__ __forceinline__ unsigned long long *cmd_word(const GridCtl &g, int pos, int x) {
    return g.cmd + (pos & (kCmdRing - 1)) * kCmdWords + x;
}
__device__ __forceinline__ unsigned long long cmd_tag(int pos) {
    return static_cast<unsigned long long>(static_cast<unsigned>(pos) + 1u) << 32;
}
__device__ __forceinline__ bool grid_failed(const GridCtl &g) {
    return __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Before a launch that begins at ring position start: an earlier launch may
// have handed out a stop there.
__global__ void k_serve_reset(GridCtl g, int start) {
    if (threadIdx.x < kCmdRing * kCmdWords) g.cmd[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        *g.done = start;
        *g.reported = start;
    }
}

// The fetching workgroup.
template <int BS>
__device__ void serve_fetch(const ServeArgs &a, const GridCtl &g, int *lds) {
    const int tid = threadIdx.x;
    long long idle0 = dev_clock();
    for (int pos = a.start;; ++pos) {
        if (tid == 0) {
            const Cmd *c = a.cmds + (pos % a.cap);
            int got = 0, failed = 0;
            for (;;) {
                const int behind = pos - __hip_atomic_load(g.reported, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (behind > 0) idle0 = dev_clock();       // work under way
                if (grid_failed(g)) { failed = 1; break; }
                if (behind < kCmdAhead &&
                    __hip_atomic_load(&c->seq, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM) == pos + 1) {
                    got = 1;
                    break;
                }
                if (dev_clock() - idle0 > a.idle_ticks) break;
                __builtin_amdgcn_s_sleep(8);
            }
            g.times[2 * (pos & (kCmdRing - 1))] = dev_clock();
            lds[CW_TYPE] = got ? __hip_atomic_load(&c->type, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) : CMD_STOP;
            if (got) {
                lds[CW_N] = __hip_atomic_load(&c->n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                lds[CW_NPAIR] = __hip_atomic_load(&c->npair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                lds[CW_SLOT] = __hip_atomic_load(&c->slot_off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                lds[CW_RID] = __hip_atomic_load(&c->rid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            lds[CW_GOT] = got;
            lds[kCmdWords] = failed;
        }
        __syncthreads();
        if (lds[kCmdWords]) return;
        const int type = lds[CW_TYPE];
        if (type == CMD_SUBMIT) {
            const int n = lds[CW_N], P = lds[CW_NPAIR];
            const SlotLayout L = slot_layout(n, P);
            int *sb = a.arena + lds[CW_SLOT];
            const int *stg = a.staging + (size_t)(pos % a.cap) * a.stage_ints;
            // (a read from host memory takes a microsecond or two: eight a thread
            // under way, where one after another a request of 64 containers and
            // all their pairs took 15 us)
            constexpr int U = 8;
            for (int base = tid; base < L.in_end; base += U * BS) {
                int v[U];
#pragma unroll
                for (int j = 0; j < U; ++j) v[j] = base + j * BS < L.in_end ? stg[base + j * BS] : 0;
#pragma unroll
                for (int j = 0; j < U; ++j)
                    if (base + j * BS < L.in_end) sb[base + j * BS] = v[j];
            }
            for (int x = tid; x < n; x += BS) {
                sb[L.host + x] = -1;
                sb[L.score + x] = 0;
            }
            for (int x = tid; x < P; x += BS) sb[L.code + x] = -1;
            if (tid == 0) {
                sb[L.failat] = -1;
                sb[L.status] = 1;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        if (tid < kCmdWords)
            __hip_atomic_store(cmd_word(g, pos, tid), cmd_tag(pos) | static_cast<unsigned>(lds[tid]), __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
        if (type == CMD_STOP) return;
        __syncthreads();                                   // lds is written again
    }
}

// The reporting workgroup: one wave.
__device__ __forceinline__ void serve_report(const ServeArgs &a, const GridCtl &g) {
    const int lane = threadIdx.x;
    int pos = a.start;
    for (;;) {
        // the next command finished, or handed out as a stop
        int state = 0;                                     // 1 finished, 2 stop, 3 stop command consumed, 4 failed
        while (!state) {
            if (__hip_atomic_load(g.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - pos > 0) {
                state = 1;
            } else {
                const unsigned long long w =
                    __hip_atomic_load(cmd_word(g, pos, CW_TYPE), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const unsigned long long got =
                    __hip_atomic_load(cmd_word(g, pos, CW_GOT), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (rec_has(w, cmd_tag(pos)) && rec_has(got, cmd_tag(pos)) && static_cast<int>(w) == CMD_STOP)
                    state = static_cast<int>(got) ? 3 : 2;
                else if (grid_failed(g))
                    state = 4;
                else
                    __builtin_amdgcn_s_sleep(4);
            }
            state = uniform(state);
        }
        if (state != 1) {
            if (lane == 0) {
                __hip_atomic_store(a.ctrl, state == 3 ? pos + 1 : pos, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(a.ctrl + 1, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            return;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        int w[kCmdWords];
#pragma unroll
        for (int x = 0; x < kCmdWords; ++x)
            w[x] = static_cast<int>(__hip_atomic_load(cmd_word(g, pos, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const int type = w[CW_TYPE], n = w[CW_N];
        const Batch b = slot_batch(a.arena + w[CW_SLOT], slot_layout(n, w[CW_NPAIR]));
        Comp *cp = a.comps + (pos % a.cap);
        if (type == CMD_SUBMIT && lane < n) {              // n <= 64
            cp->host[lane] = b.host[lane];
            cp->score[lane] = b.score[lane];
        }
        if (lane == 0) {
            cp->type = type;
            cp->rid = w[CW_RID];
            cp->n = n;
            cp->status = type == CMD_SUBMIT ? b.status[0] : 1;
            cp->failat = type == CMD_SUBMIT ? b.failat[0] : -1;
            cp->t_admit = g.times[2 * (pos & (kCmdRing - 1))];
            cp->t_decide = g.times[2 * (pos & (kCmdRing - 1)) + 1];
        }
        __threadfence_system();
        ++pos;
        if (lane == 0) {
            __hip_atomic_store(&cp->seq, pos, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(a.ctrl, pos, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(g.reported, pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int BS, int K, int CS>
__global__ __launch_bounds__(BS) void k_serve_grid(Params p, ServeArgs a, GridCtl g, long long timeout) {
    extern __shared__ __align__(16) char dsm[];
    if (static_cast<int>(blockIdx.x) >= g.wgs) {
        if (static_cast<int>(blockIdx.x) == g.wgs) serve_fetch<BS>(a, g, reinterpret_cast<int *>(dsm));
        else if (threadIdx.x < kWave) serve_report(a, g);
        return;
    }
    const Topo t = topo_of<K>(p.t);
    const GSmem sm = gcarve(dsm, t.h, t.hh, crit_count<CS>(p.m));
    int *rq_host = grid_req_lds(dsm, t.h, t.hh, crit_count<CS>(p.m));
    int *rq_cpu = rq_host + kMaxN, *rq_ram = rq_cpu + kMaxN, *rq_poff = rq_ram + kMaxN;
    int *rq_pj = rq_poff + kMaxN + 4, *rq_pbw = rq_pj + kMaxPairs, *rq_pbmax = rq_pbw + kMaxPairs;
    int *rq_cmax = rq_pbmax + kMaxPairs, *rq_rmax = rq_cmax + kMaxN;
    const bool lead = blockIdx.x == 0;
    unsigned rnd = __hip_atomic_load(g.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // selection rounds
    bool stale = true;
    long long free_at = dev_clock();                       // thread 0 of workgroup 0: the last command's end
    for (int pos = a.start;; ++pos) {
        // the command, by one thread per word
        if (threadIdx.x < kCmdWords) {
            const long long t0 = dev_clock();
            int v = 0, bad = 0;
            for (;;) {
                const unsigned long long w = __hip_atomic_load(cmd_word(g, pos, threadIdx.x), __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                if (rec_has(w, cmd_tag(pos))) {
                    v = static_cast<int>(static_cast<unsigned>(w));
                    break;
                }
                if (grid_failed(g) || dev_clock() - t0 > 2 * a.idle_ticks + timeout) {
                    __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    bad = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            sm.wst[threadIdx.x] = v;
            bad = __any(bad);
            if (threadIdx.x == 0) sm.misc[M_OK] = bad;
        }
        __syncthreads();
        const int type = sm.wst[CW_TYPE], n = sm.wst[CW_N], P = sm.wst[CW_NPAIR], off = sm.wst[CW_SLOT];
        if (sm.misc[M_OK] || type == CMD_STOP) break;
        int *sb = a.arena + off;
        const SlotLayout L = slot_layout(n, P);
        const Batch b = slot_batch(sb, L);
        if (type == CMD_SUBMIT) {
            for (int x = threadIdx.x; x <= n; x += BS) {
                rq_poff[x] = sb[L.poff + x];
                if (x < n) {
                    rq_cpu[x] = sb[L.cpu + x];
                    rq_ram[x] = sb[L.ram + x];
                    rq_cmax[x] = sb[L.cmax + x];
                    rq_rmax[x] = sb[L.rmax + x];
                    rq_host[x] = -1;
                }
            }
            for (int x = threadIdx.x; x < P; x += BS) {
                rq_pj[x] = sb[L.pj + x];
                rq_pbw[x] = sb[L.pbw + x];
                rq_pbmax[x] = sb[L.pbmax + x];
            }
            __syncthreads();
            bool placed = true;
            for (int i = 0; i < n && placed; ++i) {
                const int q0 = rq_poff[i];
                const StepIn s{0, i, n, 0, i, q0, rq_poff[i + 1] - q0, rq_cpu[i], rq_ram[i], rq_cmax[i], rq_rmax[i]};
                const ReqView rv{rq_pj + q0, rq_pbw + q0, rq_host, rq_host, rq_pbmax + q0, rq_poff, rq_pj, true};
                placed = grid_topsis_step<BS, CS>(t, p.st, p.m, b, sm, g, timeout, s, rv, p.tr, rnd, stale);
            }
            if (!placed) {
                // rejected, or a wait failed: one thread asks
                __syncthreads();
                if (threadIdx.x == 0) sm.misc[M_OK] = grid_failed(g);
                __syncthreads();
                if (sm.misc[M_OK]) break;
            }
        } else {
            // departure of an accepted request; each thread waits for its own
            // updates, whose last ones are atomics nobody else would wait for
            // before thread 0 releases them all in grid_sync
            if (lead) {
                give_back<BS>(t, p.st, b, 0, n);
                __threadfence();
            }
            stale = true;
            if (!grid_sync(g, sm.misc + M_OK, timeout)) break;
        }
        __syncthreads();
        if (lead && threadIdx.x == 0) {
            // admitted once it had been seen and the command before it was done:
            // bringing it in from host memory counts unless it passed meanwhile
            long long *at = g.times + 2 * (pos & (kCmdRing - 1));
            at[0] = max(at[0], free_at);
            at[1] = free_at = dev_clock();
            __hip_atomic_store(g.done, pos + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (lead && threadIdx.x == 0) __hip_atomic_store(g.round, rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace dcs
