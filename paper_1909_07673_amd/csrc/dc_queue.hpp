// Queue kernels of the plain form for steps spread over several workgroups:
// a whole queue of requests in one launch, TOPSIS with one workgroup per pod
// (data centers whose state does not fit one workgroup's LDS) and AHP on the
// 1-9 scale (up to 8,192 servers).  Workgroups exchange what a step needs
// through tagged words (dc_grid.hpp), with no grid barrier inside a step.
#pragma once
#include "dc_grid.hpp"

namespace dcs {

// Entry of a queue kernel.  The launch is an ordinary one, so nothing
// promises that all its workgroups run at the same time: they wait for one
// another here, before any of them has touched anything, and all leave when
// that takes longer than `patience` (the device is full of other work); the
// host then runs the queue step by step.  Once all have met they stay
// resident, so every later wait ends.  (A cooperative launch would promise
// it, but those of one process run one after another, and a serving
// session's kernel stays for as long as the session.)
// join[0] counts arrivals over all launches of the context, join[1] holds
// 2 * epoch when launch `epoch` goes ahead and 2 * epoch + 1 when it does
// not; one compare-exchange decides.
__device__ __forceinline__ bool queue_join(unsigned *join, unsigned epoch, long long patience, int *lds_flag) {
    if (threadIdx.x == 0) {
        const unsigned go = 2 * epoch, total = epoch * gridDim.x;
        const long long t0 = dev_clock();
        bool propose_go = __hip_atomic_fetch_add(join, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == total;
        unsigned d;
        for (;;) {
            d = __hip_atomic_load(join + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (d == go || d == go + 1) break;
            const bool late = dev_clock() - t0 > patience;
            if (propose_go || late) {
                (void)__hip_atomic_compare_exchange_strong(join + 1, &d, propose_go ? go : go + 1, __ATOMIC_RELAXED,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                continue;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        *lds_flag = d == go;
    }
    __syncthreads();
    return *lds_flag != 0;
}

// The request header in LDS (kReqHead ints), and the pairs of one step.
struct QueueReq {
    int *host, *cpu, *ram, *poff, *cmax, *rmax, *pj, *pbw, *pbmax;
};
constexpr int kQueueReqInts = kReqHead + 3 * kMaxN;
__device__ inline QueueReq queue_req(int *p) {
    QueueReq q;
    q.host = p;
    q.cpu = q.host + kMaxN;
    q.ram = q.cpu + kMaxN;
    q.poff = q.ram + kMaxN;
    q.cmax = q.poff + kMaxN + 4;
    q.rmax = q.cmax + kMaxN;
    q.pj = p + kReqHead;
    q.pbw = q.pj + kMaxN;
    q.pbmax = q.pbw + kMaxN;
    return q;
}

// Walks the queue: every workgroup keeps its own copy of the request's
// header, and brings in the pairs of each step one step ahead (thread x pair
// x), so that their latency passes behind the wait for the outcome of the
// step before.  step(s, rv) returns whether the container was placed.
template <int BS, class Step>
__device__ __forceinline__ void walk_queue(const Batch &b, const QueueReq &q, const GridCtl &g, int *lds_flag,
                                           Step step) {
    const int r0 = uniform(b.iroff[0]), r1 = uniform(b.iroff[1]);
    const int tid = threadIdx.x;
    for (int r = r0; r < r1; ++r) {
        const int g0 = uniform(b.coff[r]), n = uniform(b.coff[r + 1]) - g0;
        const int pb = uniform(b.poff[g0]);
        __syncthreads();                              // the last step's readers are done
        for (int x = tid; x <= n; x += BS) {
            q.poff[x] = b.poff[g0 + x] - pb;
            if (x < n) {
                q.cpu[x] = b.cpu[g0 + x];
                q.ram[x] = b.ram[g0 + x];
                q.cmax[x] = b.cmax[g0 + x];
                q.rmax[x] = b.rmax[g0 + x];
                q.host[x] = -1;
            }
        }
        __syncthreads();
        int nj = 0, nw = 0, nx = 0;                   // the next step's pairs
        for (int i = 0; i < n; ++i) {
            const int q0 = q.poff[i], P = q.poff[i + 1] - q0;
            if (tid < P) {
                q.pj[tid] = nj;
                q.pbw[tid] = nw;
                q.pbmax[tid] = nx;
            }
            if (i + 1 < n && tid < q.poff[i + 2] - q0 - P) {
                const int at = pb + q0 + P + tid;
                nj = b.pj[at];
                nw = b.pbw[at];
                nx = b.pbmax[at];
            }
            const StepIn s{r, i, n, g0, g0 + i, pb + q0, P, q.cpu[i], q.ram[i], q.cmax[i], q.rmax[i]};
            const ReqView rv{q.pj, q.pbw, q.host, q.host, q.pbmax, q.poff};
            __syncthreads();
            if (!step(s, rv)) {
                // rejected, or a wait failed: one thread asks, so that the
                // workgroup leaves or goes on as one
                __syncthreads();
                if (tid == 0) *lds_flag = __hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads();
                if (*lds_flag) return;
                break;
            }
        }
    }
}

// ---------------------------------------------------------------- TOPSIS
// One workgroup per pod, k workgroups.  K and CS as in k_topsis_grid.
template <int BS, int K, int CS>
__global__ __launch_bounds__(BS) void k_topsis_queue(Params p, GridCtl g, unsigned epoch, long long patience,
                                                     long long timeout) {
    extern __shared__ __align__(16) char dsm[];
    const Topo t = topo_of<K>(p.t);
    const GSmem sm = gcarve(dsm, t.h, t.hh, crit_count<CS>(p.m));
    if (!queue_join(g.join, epoch, patience, sm.misc + M_OK)) return;
    const QueueReq q = queue_req(grid_req_lds(dsm, t.h, t.hh, crit_count<CS>(p.m)));
    unsigned rnd = __hip_atomic_load(g.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool stale = true;
    walk_queue<BS>(p.b, q, g, sm.misc + M_OK, [&](const StepIn &s, const ReqView &rv) {
        return grid_topsis_step<BS, CS>(t, p.st, p.m, p.b, sm, g, timeout, s, rv, p.tr, rnd, stale);
    });
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(g.round, rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- AHP, 1-9 scale
// A step over gridDim.x workgroups: the first k each own a pod and compute
// its servers' criteria; C * S of them, S per criterion, turn a criterion's
// values over all servers into its local ranks (section V-B); the pods then
// sum their servers' global priorities, and the selection rounds follow.
// The values, column sums and ranks travel as 64-bit words, the 32-bit value under
// the step's tag (rec_tag), each waited for by whoever needs it.  A word of
// the next step is written only after this step's last selection round,
// whose outcome needs every pod's key, which needs every rank word, which
// needs every value word; so none is overwritten before it is read.
struct AhpGrid {
    unsigned long long *xw;   // [C][N] criterion values
    unsigned long long *zw;   // [C][N] column sums (x 2520)
    unsigned long long *lw;   // [C][N] row sums of the column-normalised matrix (FP32)
    int vmax[kMaxCrit];       // largest value of each criterion, from the capacities
    int fbytes;               // LDS of the position table, 16-byte multiple
};

// Threads per workgroup: 1,024, and 512 up to 4,096 servers (at most eight
// servers a thread): 24 arrivals at k = 20 took 2.20 ms with 1,024, 2.07 with
// 512, 2.22 with 256, the scans and barriers of the larger ones against the
// column sums of the smaller.
constexpr int kAhpQueueBlock = 1024;
constexpr int kAhpPerThread = kAhpSortMax / kAhpQueueBlock;
inline int ahp_queue_block(int N) { return N > kAhpSortMax / 2 ? kAhpQueueBlock : kAhpQueueBlock / 2; }

// Slot of the prefix sum before position q (0 <= q <= N): those behind the
// positions of a chunk of 2^lg lie together, their low bits exchanged by the
// chunk's number so that the threads' chunks start in different LDS banks;
// the one before position 0 comes first of all.
__device__ __forceinline__ int p_slot(int q, int lg) {
    const int E = 1 << lg, m = q - 1;
    return (m ^ ((m >> lg) & (E - 1))) + E;
}
__host__ __device__ inline int ahp_p_slots(int N) {
    const int E = 1 << ahp_lg_chunk(N);
    return E + ((N + E - 1) & ~(E - 1));
}

struct AhpSmem {
    GSmem g;              // tables over F; xs: feasibility row, then global priorities
    QueueReq q;
    double *scan;         // [kMaxWaves]
    unsigned *F;          // [(V + 3) / 2] positions, 16 bits each
    double *P;            // [ahp_p_slots(N)]
    double *chunk;        // [kAhpBlock] sums of chunks (over g.wst)
};

__host__ __device__ inline size_t ahp_fixed_ints(int h, int hh) {
    return 4 * (size_t)kMaxN + kStatFields * kMaxWaves + M_MISC + own_ints(h, hh) + align4(2 * (size_t)hh) + kQueueReqInts +
           2 * kMaxWaves;
}
inline size_t ahp_queue_lds(int h, int hh, int N, int fbytes) {
    const size_t tables = tab_ints(h) * sizeof(int);
    return ahp_fixed_ints(h, hh) * sizeof(int) + std::max<size_t>(tables, (size_t)fbytes + sizeof(double) * ahp_p_slots(N));
}
__device__ inline AhpSmem ahp_carve(char *base, int h, int hh, int fbytes) {
    AhpSmem s;
    s.g.pk = reinterpret_cast<int4 *>(base);
    int *p = reinterpret_cast<int *>(base) + 4 * kMaxN;
    s.g.wst = p; p += kStatFields * kMaxWaves;
    s.g.misc = p; p += M_MISC;
    s.g.own = p; p += align4(6 * (size_t)hh);
    s.g.capE = p; p += align4(h);
    s.g.xs = p; p += align4(2 * (size_t)hh);
    s.q = queue_req(p); p += kQueueReqInts;
    s.scan = reinterpret_cast<double *>(p); p += 2 * kMaxWaves;
    (void)carve_tabs(s.g, p, h);
    s.F = reinterpret_cast<unsigned *>(p);
    s.P = reinterpret_cast<double *>(reinterpret_cast<char *>(p) + fbytes);
    static_assert(kAhpBlock * sizeof(double) <= kStatFields * kMaxWaves * sizeof(int), "chunk sums over the statistics slots");
    s.chunk = reinterpret_cast<double *>(s.g.wst);
    return s;
}

// DPP moves and lane reads of a 32- or 64-bit value.
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T dpp_zero(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp<CTRL, ROWS>(0, __builtin_bit_cast(int, v)));
    } else {
        const long long x = __builtin_bit_cast(long long, v);
        const unsigned lo = dpp<CTRL, ROWS>(0, static_cast<int>(x)), hi = dpp<CTRL, ROWS>(0, static_cast<int>(x >> 32));
        return __builtin_bit_cast(T, static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
    }
}
template <class T>
__device__ __forceinline__ T read_lane(T v, int lane) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
    } else {
        const long long x = __builtin_bit_cast(long long, v);
        const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(x), lane);
        const unsigned hi = __builtin_amdgcn_readlane(static_cast<int>(x >> 32), lane);
        return __builtin_bit_cast(T, static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
    }
}

// Exclusive scan of one value per thread over the block, total its sum: a
// DPP scan of each wave, the wave sums through LDS (slots: one per wave) and
// one more DPP scan of them in every wave.  One barrier; slots must not be
// written again before another.
template <int BS, class T>
__device__ __forceinline__ T block_scan(T v, T *slots, T &total) {
    static_assert(BS / kWave <= 16, "the wave sums are scanned within one DPP row");
    const int lane = threadIdx.x & (kWave - 1), wid = uniform(threadIdx.x / kWave);
    T inc = v;
    inc += dpp_zero<0x111, 0xf>(inc);
    inc += dpp_zero<0x112, 0xf>(inc);
    inc += dpp_zero<0x114, 0xf>(inc);
    inc += dpp_zero<0x118, 0xf>(inc);
    inc += dpp_zero<0x142, 0xa>(inc);
    inc += dpp_zero<0x143, 0xc>(inc);
    if (lane == kWave - 1) slots[wid] = inc;
    __syncthreads();
    T w = lane < BS / kWave ? slots[lane] : T(0);
    w += dpp_zero<0x111, 0xf>(w);
    w += dpp_zero<0x112, 0xf>(w);
    w += dpp_zero<0x114, 0xf>(w);
    w += dpp_zero<0x118, 0xf>(w);
    total = read_lane(w, BS / kWave - 1);
    const T before = wid ? read_lane(w, wid - 1) : T(0);
    return before + (inc - v);
}

// Sum of the chunks before chunk 64 wid + lane, by the tree of
// block_excl_scan<kAhpBlock> over the chunk sums sh: a wave holds all of them,
// four neighbours a lane, so that the eight distances need no barrier.
__device__ __forceinline__ double chunks_before(const double *sh, int wid) {
    static_assert(kAhpBlock == 4 * kWave, "four chunks a lane");
    const int lane = threadIdx.x & (kWave - 1);
    double a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = sh[4 * lane + j];
    // distances 1 and 2: a neighbour's or the next lane's (wave_shr:1)
    const double p3 = dpp_zero<0x138, 0xf>(a[3]);
    a[3] += a[2]; a[2] += a[1]; a[1] += a[0]; a[0] += p3;
    const double q2 = dpp_zero<0x138, 0xf>(a[2]), q3 = dpp_zero<0x138, 0xf>(a[3]);
    a[3] += a[1]; a[2] += a[0]; a[1] += q3; a[0] += q2;
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) {              // distances 4 s
        double o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            o[j] = s == 1 ? dpp_zero<0x138, 0xf>(a[j])
                 : s == 2 ? dpp_zero<0x138, 0xf>(dpp_zero<0x138, 0xf>(a[j])) : __shfl_up(a[j], s);
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] += lane >= s ? o[j] : 0.0;
    }
    const int t = wid * kWave + lane - 1, src = max(t, 0) >> 2;
    double r = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double o = __shfl(a[j], src);
        r = t >= 0 && (t & 3) == j ? o : r;
    }
    return r;
}

// The bounds of saaty_buckets for a value v, looked up: at(t) is the number
// of values below t (0 <= t <= V + 1).  2v < 2^18, so the divisions by
// 3, 5, .. 17 go through FP32 reciprocals (fdiv).
template <class At>
__device__ __forceinline__ SaatyBuckets saaty_positions(int v, int V, int n, At at) {
    SaatyBuckets b;
    b.lv = at(v);
    b.uv = at(v + 1);
    b.ai[1] = b.uv;
    b.bi[1] = b.lv;
#pragma unroll
    for (int k = 2; k <= 9; ++k) {
        b.ai[k] = at(min(max(((2 * k - 1) * v + 1) >> 1, v + 1), V + 1));
        b.bi[k] = at(min(fdiv(2 * v, 1.0f / (2 * k - 1)) + 1, v));
    }
    b.ai[10] = n;
    b.bi[10] = 0;
    return b;
}

// Thread: the 32-bit values of the tagged words at(e) for every e of the bits
// of todo, once each carries the tag; only the words still missing are read
// again.  False when the wait timed out or a workgroup reported an error.
template <int E, class At>
__device__ __forceinline__ bool words_get(const GridCtl &g, unsigned todo, At at, unsigned long long tag,
                                          long long timeout, int (&v)[E]) {
    const long long t0 = dev_clock();
    while (todo) {
        unsigned long long w[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (todo >> e & 1) w[e] = __hip_atomic_load(at(e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((todo >> e & 1) && rec_has(w[e], tag)) {
                v[e] = static_cast<int>(static_cast<unsigned>(w[e]));
                todo &= ~(1u << e);
            }
        if (!todo) break;
        if (__hip_atomic_load(g.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || dev_clock() - t0 > timeout) {
            __hip_atomic_store(g.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// Servers from which a criterion's column sums are shared out over its
// slices: each thread then computes one and reads the others' from their
// words, which costs one more exchange (about 2 us) and saves 1.1 us per
// column the thread would take otherwise.
constexpr int kAhpSplitColumns = 3 * kAhpQueueBlock;

// Local ranks of criterion c for slice s of S (servers [s R, (s + 1) R)).
// A criterion's values are bounded by its capacity, so counting takes the
// place of a sort: F[t], the number of servers with a value below t, from a
// histogram in LDS and one scan; every bucket bound of saaty_sum is then one
// LDS read (the sorted form took 13 dependent reads per bound).  Column sums
// are exact integers as before.  Where the values of a criterion fill more
// bins than LDS holds (capacities past some 40,000 at 8,192 servers) the
// sorted passes remain.  The prefix sums of 1 / column sum take one term per
// server in the order of those passes, so the scores do not depend on which of
// the two ran: 1.2 to 1.5 us of a step (of 30 at 8,192 servers, 22 at 2,000)
// more than a block scan of one term per distinct value, whose other order of
// additions rounded a row sum in some 10^9 to the next FP32 value.
template <int BS>
__device__ __forceinline__ bool ahp_local_rank(const AhpSmem &sm, const AhpGrid &a, const GridCtl &g, int N, int c,
                                               bool cost, int s, int S, unsigned long long tag, long long timeout) {
    constexpr int E = kAhpPerThread;
    const int tid = threadIdx.x, V = a.vmax[c];
    const unsigned long long *xw = a.xw + static_cast<size_t>(c) * N;
    unsigned short *F16 = reinterpret_cast<unsigned short *>(sm.F);
    unsigned *H = reinterpret_cast<unsigned *>(sm.P);
    // few values would meet on few LDS words: their histogram takes several
    // copies, in the space of P
    const int slots = 2 * ahp_p_slots(N);
    int lg = 3;
    while (lg > 0 && ((V + 1) << lg) > slots) --lg;
    const bool copies = lg >= 2;
    // clear, while the values come in
    const int fw = (V + 3) >> 1;
    if (copies) {
        for (int x = tid; x < (V + 1) << lg; x += BS) H[x] = 0;
    } else {
        for (int x = tid; x < fw; x += BS) sm.F[x] = 0;
    }
    // the values: server e * BS + tid in v[e], this slice's row in v[E]
    const int R = (N + S - 1) / S, row = s * R + tid;
    const bool has_row = tid < R && row < N;
    int v[E + 1] = {};
    unsigned mine = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) mine |= e * BS + tid < N ? 1u << e : 0u;
    bool bad = !words_get<E + 1>(g, mine | (has_row ? 1u << E : 0u),
                                 [&](int e) { return xw + (e < E ? e * BS + tid : row); }, tag, timeout, v);
    if (bad) sm.g.misc[M_OK] = 1;
    __syncthreads();
    if (sm.g.misc[M_OK]) return false;
    // histogram; where a wave's values repeat (path bandwidths capped by one
    // peer's uplink), the servers with its first lane's value count as one.
    // What is counted before a server among those of its value goes above its
    // value (V < 2^17, N < 2^14; an array of its own would spill)
    const int copy = tid & ((1 << lg) - 1), lane = tid & (kWave - 1);
    auto val = [&](int e) { return v[e] & 0x1ffff; };
    auto pos = [&](int e) { return static_cast<int>(static_cast<unsigned>(v[e]) >> 17); };
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e * BS >= N) continue;
        const bool in = e * BS + tid < N;
        unsigned was = 0;
        if (copies) {
            if (in) was = atomicAdd(H + (v[e] << lg) + copy, 1u);
        } else {
            const int half = 16 * (v[e] & 1);
            const bool same = in && v[e] == uniform(v[e]);
            const unsigned long long m = __ballot(same);
            const bool first = same && lane == __builtin_ctzll(m);
            const unsigned cnt = first ? static_cast<unsigned>(__builtin_popcountll(m)) : 1u;
            if (in && (!same || first)) was = atomicAdd(sm.F + (v[e] >> 1), cnt << half) >> half & 0xffffu;
        }
        v[e] |= static_cast<int>(was << 17);
    }
    if (!copies) {
        // (apart, so that all additions are under way before one is waited for)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e * BS >= N) continue;
            const bool same = e * BS + tid < N && val(e) == uniform(val(e));
            const unsigned long long m = __ballot(same);
            const int group = __builtin_amdgcn_readlane(pos(e), m ? __builtin_ctzll(m) : 0);
            const unsigned ahead = __builtin_amdgcn_mbcnt_hi(m >> 32, __builtin_amdgcn_mbcnt_lo(m, 0));
            if (same) v[e] = val(e) | static_cast<int>((group + ahead) << 17);
        }
    }
    __syncthreads();
    if (copies) {
        // a value's copies, each left with the count of those before it
        for (int x = tid; x < 2 * fw; x += BS) {
            unsigned cnt = 0;
            if (x <= V) {
                unsigned h[8];
#pragma unroll
                for (int y = 0; y < 8; ++y) h[y] = y < 1 << lg ? H[(x << lg) + ((y + tid) & ((1 << lg) - 1))] : 0u;
#pragma unroll
                for (int y = 0; y < 8; ++y) {
                    if (y < 1 << lg) H[(x << lg) + ((y + tid) & ((1 << lg) - 1))] = cnt;
                    cnt += h[y];
                }
            }
            F16[x] = static_cast<unsigned short>(cnt);
        }
        __syncthreads();
    }
    // counts to positions: each thread scans an odd number of words, so the
    // threads' runs start in different banks
    {
        const int per = ((fw + BS - 1) / BS) | 1, w0 = min(fw, tid * per), w1 = min(fw, w0 + per);
        constexpr int U = 8;                           // words in flight
        int sum = 0;
        for (int x = w0; x < w1; x += U) {
            unsigned o[U];
#pragma unroll
            for (int j = 0; j < U; ++j) o[j] = x + j < w1 ? sm.F[x + j] : 0u;
#pragma unroll
            for (int j = 0; j < U; ++j) sum += static_cast<int>((o[j] & 0xffffu) + (o[j] >> 16));
        }
        int total;
        unsigned at = block_scan<BS>(sum, reinterpret_cast<int *>(sm.scan), total);
        for (int x = w0; x < w1; x += U) {
            unsigned o[U];
#pragma unroll
            for (int j = 0; j < U; ++j) o[j] = x + j < w1 ? sm.F[x + j] : 0u;
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const unsigned hi = at + (o[j] & 0xffffu);
                if (x + j < w1) sm.F[x + j] = at | hi << 16;
                at = hi + (o[j] >> 16);
            }
        }
    }
    __syncthreads();
    auto F = [&](int t) { return static_cast<int>(F16[t]); };
    // each server's position in ascending order (equal values in any order:
    // their terms are the same), and at each position 1 / column sum
    const int lgE = ahp_lg_chunk(N);
    auto positions = [&]() {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e * BS + tid < N)
                v[e] += static_cast<int>(F(val(e)) + (copies ? H[(val(e) << lg) + copy] : 0u)) << 17;
        if (copies) __syncthreads();                      // H makes room for P
    };
    SaatyBuckets rb;
    if (N > kAhpSplitColumns) {
        unsigned long long *zw = a.zw + static_cast<size_t>(c) * N;
        if (has_row) {
            rb = saaty_positions(v[E], V, N, F);
            const int cs = saaty_sum<int>(rb, N, cost, [](int lo, int hi) { return hi - lo; });
            __hip_atomic_store(zw + row, tag | static_cast<unsigned>(cs), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        positions();
        int z[E];
        bad = !words_get<E>(g, mine, [&](int e) { return zw + e * BS + tid; }, tag, timeout, z);
        if (bad) sm.g.misc[M_OK] = 1;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (!bad && e * BS + tid < N) sm.P[p_slot(pos(e) + 1, lgE)] = 1.0 / static_cast<double>(z[e]);
    } else {
        positions();
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e * BS + tid < N) {
                const SaatyBuckets b = saaty_positions(val(e), V, N, F);
                const int cs = saaty_sum<int>(b, N, cost, [](int lo, int hi) { return hi - lo; });
                sm.P[p_slot(pos(e) + 1, lgE)] = 1.0 / static_cast<double>(cs);
            }
        rb = saaty_positions(v[E], V, N, F);
    }
    if (tid == 0) sm.P[0] = 0.0;
    __syncthreads();
    if (sm.g.misc[M_OK]) return false;
    // prefix sums, in the order of k_ahp_sort_row: four waves take a chunk a
    // thread
    {
        const int len = min(N, (tid + 1) << lgE) - (tid << lgE), swap = tid & ((1 << lgE) - 1);
        double *chunk = sm.P + ((tid + 1) << lgE);        // slot of the chunk's first
        constexpr int U = 8;                              // terms in flight
        if (tid < kAhpBlock) {
            double run = 0.0;
            for (int m = 0; m < len; m += U) {
                double d[U];
#pragma unroll
                for (int j = 0; j < U; ++j) d[j] = m + j < len ? chunk[(m + j) ^ swap] : 0.0;
#pragma unroll
                for (int j = 0; j < U; ++j) run += d[j];
            }
            sm.chunk[tid] = run;
        }
        __syncthreads();
        if (tid < kAhpBlock) {
            double run = chunks_before(sm.chunk, uniform(tid / kWave));
            for (int m = 0; m < len; m += U) {
                double d[U];
#pragma unroll
                for (int j = 0; j < U; ++j) d[j] = m + j < len ? chunk[(m + j) ^ swap] : 0.0;
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    run += d[j];
                    if (m + j < len) chunk[(m + j) ^ swap] = run;
                }
            }
        }
    }
    __syncthreads();
    if (has_row) {
        const double r = saaty_sum<double>(
            rb, N, !cost, [&](int lo, int hi) { return sm.P[p_slot(hi, lgE)] - sm.P[p_slot(lo, lgE)]; });
        __hip_atomic_store(a.lw + static_cast<size_t>(c) * N + row, tag | __float_as_uint(static_cast<float>(r)),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
}

template <int BS>
__device__ __forceinline__ bool grid_ahp_step(const Params &p, const Topo &t, const AhpSmem &sm, const AhpGrid &a,
                                              const GridCtl &g, long long timeout, const StepIn &s, const ReqView &rv,
                                              unsigned &rnd, bool &stale) {
    const int w = blockIdx.x, h = t.h, hh = t.hh, nc = p.m.nc, N = t.N, ubase = w * hh, P = s.P;
    const bool pod = w < t.k;
    const unsigned long long tag = rec_tag(rnd);
    int *feas = sm.g.xs;
    float *pg = reinterpret_cast<float *>(sm.g.xs + hh);
    if (pod) {
        int slot = -1;
        if (w == 0 && threadIdx.x == 0) {
            if (s.i == 0) p.b.tsb[s.r] = dev_clock();
            if (p.tr.stride > 0) slot = trace_slot(p.tr, 0, p.b.rid[s.r], s.i);
        }
        grid_criteria<BS, 0>(t, p.st, p.m, sm.g, s, rv, stale, [&](int x, int f, auto get) {
            feas[x] = f;
#pragma unroll
            for (int c = 0; c < kMaxCrit; ++c) {
                if (c >= nc) break;
                __hip_atomic_store(a.xw + static_cast<size_t>(c) * N + ubase + x, tag | static_cast<unsigned>(get(c)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        });
        for (int e = threadIdx.x; e < h; e += BS) rec_put(g, w, kRecCapE + e, tag, sm.g.capE[e]);
        if (threadIdx.x == 0) {
            rec_put(g, w, kRecCapP, tag, sm.g.misc[M_CAPP]);
            if (w == 0) rec_put(g, 0, kRecTrace, tag, slot);
        }
        __syncthreads();                                  // the tables make room for F
    } else {
        if (threadIdx.x == 0) sm.g.misc[M_OK] = 0;
        __syncthreads();
    }
    const int S = gridDim.x / nc, c = w % nc, sl = w / nc;
    if (sl < S && !ahp_local_rank<BS>(sm, a, g, N, c, p.m.cost[c] != 0, sl, S, tag, timeout)) return false;
    if (pod) {
        bool bad = false;
        if (static_cast<int>(threadIdx.x) < P) {
            const int4 me = sm.g.pk[threadIdx.x];
            const int e = me.y & 0xffff, d = me.y >> 16;
            const int ws[2] = {e / h, d}, xs[2] = {kRecCapE + e % h, kRecCapP};
            int cv[2];
            bad = !rec_get(g, 2, ws, xs, tag, timeout, cv);
            grid_deficits(sm.g, P, me, cv[0], cv[1]);
        }
        int slot = -1;
        if (p.tr.stride > 0) {
            const int zw[1] = {0}, zx[1] = {kRecTrace};
            int zv[1];
            bad |= !rec_get(g, 1, zw, zx, tag, timeout, zv);
            slot = zv[0];
        }
        // global priorities of the pod's servers, as k_ahp_pg sums them
        const double invN = 1.0 / N;
        for (int x = threadIdx.x; x < hh; x += BS) {
            int l[kMaxCrit] = {};
            bad |= !words_get<kMaxCrit>(g, (1u << nc) - 1, [&](int q) { return a.lw + static_cast<size_t>(q) * N + ubase + x; },
                                        tag, timeout, l);
            double sum = 0.0;
#pragma unroll
            for (int q = 0; q < kMaxCrit; ++q)
                if (q < nc) sum += p.p1[q] * (static_cast<double>(__int_as_float(l[q])) * invN);
            pg[x] = static_cast<float>(sum);
            if (slot >= 0) p.tr.scores[static_cast<size_t>(slot) * N + ubase + x] = pg[x];
        }
        if (bad) sm.g.misc[M_OK] = 1;
        __syncthreads();
        if (sm.g.misc[M_OK]) return false;
    }
    const Deficits df = read_deficits(sm.g);
    return grid_select<BS, false>(t, p.st, p.m, p.b, sm.g, g, timeout, s, rv, rnd, stale, pod ? hh : 0, feas,
                           [&](int x) -> unsigned long long {
                               if (!feas[x] || !(p.m.route_end || deficits_allow(t, df, w, x))) return 0ull;
                               return score_key(pg[x], ubase + x);
                           });
}

template <int BS>
__global__ __launch_bounds__(BS) void k_ahp_queue(Params p, GridCtl g, AhpGrid a, unsigned epoch, long long patience,
                                                  long long timeout) {
    extern __shared__ __align__(16) char dsm[];
    const Topo t = p.t;
    const AhpSmem sm = ahp_carve(dsm, t.h, t.hh, a.fbytes);
    if (!queue_join(g.join, epoch, patience, sm.g.misc + M_OK)) return;
    unsigned rnd = __hip_atomic_load(g.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool stale = true;
    walk_queue<BS>(p.b, sm.q, g, sm.g.misc + M_OK, [&](const StepIn &s, const ReqView &rv) {
        return grid_ahp_step<BS>(p, t, sm, a, g, timeout, s, rv, rnd, stale);
    });
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(g.round, rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace dcs
