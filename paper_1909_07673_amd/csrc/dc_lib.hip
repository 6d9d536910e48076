// libdcsched host runtime: the C ABI of include/dcsched.h over the kernels of
// dc_kernels.hpp, dc_grid.hpp, dc_queue.hpp, dc_ahp_large.hpp, dc_serve.hpp
// and dc_tiles.hpp.  Owns the device-resident data-center state, uploads
// request batches, drives the plain (a queue in one launch, or one launch per
// step or stage), batched (one persistent launch over all instances) and
// serving (one persistent launch fed through a ring) forms, and collects
// results.
#include "../../include/dcsched.h"
#include "dc_kernels.hpp"
#include "dc_grid.hpp"
#include "dc_queue.hpp"
#include "dc_ahp_large.hpp"
#include "dc_tiles.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <chrono>
#include <fstream>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

using namespace dcs;

namespace {

// Launch shape of the batched kernel: threads per workgroup, servers each
// thread scores together, peers whose path tables are built together.
struct Shape {
    int bs = 1024, g = 1, pc = 1;
    bool operator==(const Shape &o) const { return bs == o.bs && g == o.g && pc == o.pc; }
};

// (threads, servers per thread) pairs the batched kernel is built for.
constexpr int kBatchedShapes[][2] = {{256, 1}, {256, 2}, {256, 4}, {512, 1}, {512, 2}, {512, 4}, {1024, 1}, {1024, 2}};

bool batched_shape_built(int bs, int g) {
    for (const auto &x : kBatchedShapes)
        if (x[0] == bs && x[1] == g) return true;
    return false;
}

// A request's containers and edges as submitted, kept so that what each
// unit and unit pair is given can be handed back to them.
struct Members {
    std::vector<int> cpu, cmax, ram, rmax;   // per container: demand intervals
    std::vector<int> emin, emax;             // per edge: bandwidth interval
    std::vector<int> epair;                  // per edge: the unit pair carrying it (unit CSR index), -1 inside a unit
};

// A request as the device schedules it.  Containers of a pod share one
// server (section II-A, Eq. (8)), so the unit of placement is the pod: one
// unit per pod, in the order of each pod's first container (a container
// without a pod is a pod of its own), asking for the summed CPU and RAM of
// its containers.  The peers of unit g are the earlier units h whose
// containers exchange traffic with g's, each with the summed demand: the two
// pods sit on one server each, so their links share one route.  Traffic
// inside a pod needs no network.  Without pods every container is a unit
// and its peers are the earlier containers it talks to.  Demands are
// intervals (section II-A); minima and maxima are summed separately.
struct Units {
    int n = 0;                         // containers
    std::vector<int> cpu, ram;         // per unit, minima
    std::vector<int> cmax, rmax;       // per unit, maxima
    std::vector<int> poff, pj, pbw;    // peers of each unit (CSR), ascending unit index, minimum demand
    std::vector<int> pbmax;            // maximum demand of each peer pair
    std::vector<int> unit_of;          // container -> unit
    std::vector<int> first;            // unit -> its smallest container index
    Members mem;
    int nu() const { return (int)cpu.size(); }
};

// Builds the units of a validated request; DC_EINVAL when a summed demand
// reaches past the 2^22 bound of capacities.  pod[i] >= 0 names container
// i's pod (equal ids, same pod); pod[i] < 0 or pod == NULL: no pod.
// cpu_max, ram_max, bw_max (per edge) are the maxima, or NULL for fixed
// demands.
int build_units(int n, const int *cpu, const int *cpu_max, const int *ram, const int *ram_max, int m,
                const int *edges, const int *bw_max, const int *pod, Units &u) {
    constexpr long long kCap = 1LL << 22;
    u = Units{};
    u.n = n;
    u.unit_of.assign(n, -1);
    std::vector<long long> uc, ur, ucx, urx;
    std::map<int, int> pod_unit;
    Members &M = u.mem;
    for (int i = 0; i < n; ++i) {
        int g = -1;
        if (pod && pod[i] >= 0) {
            auto it = pod_unit.find(pod[i]);
            if (it != pod_unit.end()) g = it->second;
            else pod_unit[pod[i]] = g = (int)uc.size();
        } else {
            g = (int)uc.size();
        }
        if (g == (int)uc.size()) {
            uc.push_back(0);
            ur.push_back(0);
            ucx.push_back(0);
            urx.push_back(0);
            u.first.push_back(i);
        }
        u.unit_of[i] = g;
        M.cpu.push_back(cpu[i]);
        M.ram.push_back(ram[i]);
        M.cmax.push_back(cpu_max ? cpu_max[i] : cpu[i]);
        M.rmax.push_back(ram_max ? ram_max[i] : ram[i]);
        uc[g] += cpu[i];
        ur[g] += ram[i];
        ucx[g] += M.cmax.back();
        urx[g] += M.rmax.back();
    }
    const int nu = (int)uc.size();
    for (int g = 0; g < nu; ++g) {
        if (ucx[g] > kCap || urx[g] > kCap) return DC_EINVAL;
        u.cpu.push_back((int)uc[g]);
        u.ram.push_back((int)ur[g]);
        u.cmax.push_back((int)ucx[g]);
        u.rmax.push_back((int)urx[g]);
    }
    std::vector<long long> bw((size_t)nu * nu, 0), bwx((size_t)nu * nu, 0);
    for (int q = 0; q < m; ++q) {
        const int a = u.unit_of[edges[3 * q]], b = u.unit_of[edges[3 * q + 1]];
        M.emin.push_back(edges[3 * q + 2]);
        M.emax.push_back(bw_max ? bw_max[q] : edges[3 * q + 2]);
        if (a == b) continue;
        bw[(size_t)a * nu + b] += edges[3 * q + 2];
        bw[(size_t)b * nu + a] += edges[3 * q + 2];
        bwx[(size_t)a * nu + b] += M.emax.back();
        bwx[(size_t)b * nu + a] += M.emax.back();
    }
    std::vector<int> pidx((size_t)nu * nu, -1);
    u.poff.assign(1, 0);
    for (int g = 0; g < nu; ++g) {
        for (int h = 0; h < g; ++h) {
            const long long w = bw[(size_t)g * nu + h], wx = bwx[(size_t)g * nu + h];
            if (wx > kCap) return DC_EINVAL;
            if (w > 0) {
                pidx[(size_t)g * nu + h] = pidx[(size_t)h * nu + g] = (int)u.pj.size();
                u.pj.push_back(h);
                u.pbw.push_back((int)w);
                u.pbmax.push_back((int)wx);
            }
        }
        u.poff.push_back((int)u.pj.size());
    }
    for (int q = 0; q < m; ++q)
        M.epair.push_back(pidx[(size_t)u.unit_of[edges[3 * q]] * nu + u.unit_of[edges[3 * q + 1]]]);
    return DC_OK;
}

// Hands the allocation a of a unit (or unit pair) back to its members who[]
// in order: each first gets its minimum, then what is left goes up to each
// one's maximum in turn.
void hand_back(long long a, const std::vector<int> &who, const std::vector<int> &mn, const std::vector<int> &mx,
               int32_t *out) {
    for (int x : who) { out[x] = mn[x]; a -= mn[x]; }
    for (int x : who) {
        const long long t = std::min<long long>(a, (long long)mx[x] - mn[x]);
        out[x] += (int32_t)t;
        a -= t;
    }
}

// Allocations per container and per edge from those of the units (ua_cpu,
// ua_ram, nu entries) and unit pairs (pa, relative to the request's first
// pair).  An edge inside a unit uses no link and gets its maximum.
void members_alloc(const Members &M, const std::vector<int> &unit_of, int nu, const int *ua_cpu,
                   const int *ua_ram, const int *pa, int32_t *cpu, int32_t *ram, int32_t *bw) {
    const int n = (int)M.cpu.size(), m = (int)M.emin.size();
    std::vector<std::vector<int>> who(nu);
    for (int i = 0; i < n; ++i) who[unit_of[i]].push_back(i);
    for (int g = 0; g < nu; ++g) {
        if (cpu) hand_back(ua_cpu[g], who[g], M.cpu, M.cmax, cpu);
        if (ram) hand_back(ua_ram[g], who[g], M.ram, M.rmax, ram);
    }
    if (!bw) return;
    std::map<int, std::vector<int>> by_pair;
    for (int q = 0; q < m; ++q) {
        if (M.epair[q] < 0) bw[q] = M.emax[q];
        else by_pair[M.epair[q]].push_back(q);
    }
    for (const auto &kv : by_pair) hand_back(pa[kv.first], kv.second, M.emin, M.emax, bw);
}

// One uploaded set of requests (the pending queue at a dc_schedule call).
struct DevBatch {
    int R = 0, Ct = 0, Pt = 0, I = 0;
    int *dmem = nullptr;           // device: inputs then outputs
    size_t in_ints = 0, out_ints = 0;
    Batch view{};
    std::vector<int64_t> ids;      // request id per batch request
    std::vector<int> inst, coff, poff, pj, pbw, cpu, ram, iroff;   // unit level (coff: units per request)
    std::vector<int> cmax, rmax, pbmax;                            // unit level maxima
    std::vector<Members> mem;                                      // per request
    size_t o_alloc = 0;                                            // output offset of cpua, rama, pbwa
    std::vector<int> cnt, cuoff, unit_of, first;                   // containers per request, their units, first containers
    std::vector<int> host, status, failat;
    std::vector<float> score;
    std::vector<long long> tsb, tse;
    hipGraphExec_t gexec = nullptr;    // batched form: captured launch of this batch
    Shape gshape{0, 0, 0};             // launch shape it was captured with
    ~DevBatch() {
        if (gexec) (void)hipGraphExecDestroy(gexec);
    }
};

struct ReqLoc {
    int batch = -1, r = -1;
    bool released = false;
};

// Serving form: one live request's slot in the device arena.
struct ServeSlot {
    size_t off = 0, ints = 0;      // offset and size in the arena (int32 units)
    int n = 0, P = 0;              // units and peer pairs as the device sees them
    int nc = 0;                    // containers
    std::vector<int> unit_of, first;
    Members mem;
    int status = -1;               // -1 pending, 1 accepted, 0 rejected
    bool released = false;
    std::vector<int> hosts;        // attempt record from the completion
};

// Serving form state: rings in coherent pinned host memory, the device slot
// arena with a first-fit allocator, and the host's ring positions.
struct Serve {
    Cmd *cmds = nullptr;
    Comp *comps = nullptr;
    int *ctrl = nullptr;
    int *staging = nullptr;
    int *arena = nullptr;
    size_t arena_ints = 0;
    std::map<size_t, size_t> free_list;     // offset -> size, int32 units
    int cap = 1024, stage_ints = 0, bs = 1024, pc = 1;
    size_t lds = 0;
    long long idle_ticks = 100000000LL;     // 1 s of device clock
    int64_t host_pos = 0, comp_pos = 0;     // commands published / completions consumed
    std::unordered_map<int64_t, ServeSlot> slots;
    std::unordered_map<int, int64_t> rid_to_id;
    std::vector<std::pair<int64_t, float>> service_us;
    hipStream_t aux = nullptr;              // copies while the persistent kernel runs
    bool launched = false;
};

bool serve_alloc(Serve &sv, size_t ints, size_t *off) {
    ints = (ints + 3) & ~size_t(3);
    for (auto it = sv.free_list.begin(); it != sv.free_list.end(); ++it) {
        if (it->second >= ints) {
            *off = it->first;
            const size_t rest = it->second - ints, roff = it->first + ints;
            sv.free_list.erase(it);
            if (rest) sv.free_list[roff] = rest;
            return true;
        }
    }
    return false;
}

void serve_free(Serve &sv, size_t off, size_t ints) {
    ints = (ints + 3) & ~size_t(3);
    auto it = sv.free_list.emplace(off, ints).first;
    auto nx = std::next(it);
    if (nx != sv.free_list.end() && it->first + it->second == nx->first) {
        it->second += nx->second;
        sv.free_list.erase(nx);
    }
    if (it != sv.free_list.begin()) {
        auto pv = std::prev(it);
        if (pv->first + pv->second == it->first) {
            pv->second += it->second;
            sv.free_list.erase(it);
        }
    }
}

}  // namespace

struct dc_ctx {
    dc_config cfg{};
    Topo t{};
    Method m{};
    int N = 0, I = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    bool poisoned = false;
    int *d_state = nullptr;        // [I][6][N]
    int *d_init = nullptr;         // [I][6][N]
    int *d_xs = nullptr;           // [I][nc+6][N]
    int *d_colpart = nullptr;      // AHP [nc][nI][N]
    float *d_rowpart = nullptr;    // AHP [nc][nJ][N]
    int ti = 0, tj = 0, nI = 0, nJ = 0;
    bool ahp_sorted = false;       // AHP on the 1-9 scale through the sorted passes
    int *d_ysort = nullptr;        // [nc][N]
    int *d_runs = nullptr;         // [nc][sort_runs][1024] sorted runs before their merge
    double *d_wsort = nullptr;     // [nc][N]
    int sort_runs = 1;             // sorted passes: runs of 1,024 values sorted apart, then merged
    int *d_tmeta = nullptr, *d_tcount = nullptr;
    float *d_tscore = nullptr;
    int plain_bs = 1024;
    Shape bshape{};                // batched form: current launch shape
    int pc_plain = 1, pc_batched = 1;  // peer chunk of the plain form; largest the batched LDS holds
    bool plain_res = false;        // plain kernel stages state + scratch in LDS
    size_t lds_plain = 0, lds_select = 0;
    std::vector<std::unique_ptr<DevBatch>> batches;
    // the batches' device memory, cut from slabs (freed with the context),
    // and a pinned buffer for what goes up and comes back: an allocation for
    // each would cost a small call more than its kernel
    std::vector<int *> slabs;
    size_t slab_at = 0, slab_end = 0;      // free part of the last slab (int32 units)
    int *pinned = nullptr;
    size_t pinned_ints = 0;
    std::vector<int> queued;       // batches uploaded and waiting to run
    std::vector<int> pend_inst;
    std::vector<Units> pend_units;
    std::vector<int64_t> pend_ids;
    std::unordered_map<int64_t, ReqLoc> loc;
    int64_t next_id = 0;
    std::vector<dc_result> ready;  // decided results not yet handed out, from ready_head on
    size_t ready_head = 0;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    float last_ms = 0.f;
    int64_t last_launches = 0, last_steps = 0;
    std::unique_ptr<Serve> sv;     // serving form only
    // cooperative (one workgroup per pod) TOPSIS step
    bool use_grid = false;
    GridCtl grid{};
    int *d_grid = nullptr;         // backing allocation of grid
    size_t lds_grid = 0;
    long long grid_timeout = 10000000LL;   // 100 ms of device clock per barrier wait
    // plain form: a queue in one launch over several workgroups
    enum { QUEUE_NONE, QUEUE_TOPSIS, QUEUE_AHP };
    int queue = QUEUE_NONE;
    int queue_wgs = 0;
    size_t lds_queue = 0;
    unsigned epoch = 0;            // launches of the queue kernel
    long long patience = 2000000LL;        // 20 ms of device clock for its workgroups to meet
    AhpGrid ahp{};
    bool ahp_large = false;        // AHP on the 1-9 scale past the sorted passes, by distinct value
    AhpLarge large{};
    void *d_large = nullptr;
    size_t lds_count = 0;
    hipError_t launch_err = hipSuccess;    // first failed cooperative launch of a run
    hipStream_t cap_stream = nullptr;      // graph capture (batched form)
};

#define HIPCHK(expr)                                       \
    do {                                                   \
        hipError_t e_ = (expr);                            \
        if (e_ != hipSuccess) {                            \
            ctx->poisoned = true;                          \
            std::fprintf(stderr, "libdcsched: %s failed: %s\n", #expr, hipGetErrorString(e_)); \
            return DC_EDEVICE;                             \
        }                                                  \
    } while (0)

namespace {

int check_config(const dc_config *c) {
    if (!c) return DC_EINVAL;
    if (c->k < 4 || c->k > 64 || (c->k & 1)) return DC_EINVAL;
    if (c->n_instances < 1 || c->n_instances > 65536) return DC_EINVAL;
    if (c->mode < DC_MODE_PLAIN || c->mode > DC_MODE_SERVING) return DC_EINVAL;
    if (c->method != DC_TOPSIS && c->method != DC_AHP) return DC_EINVAL;
    if (c->method == DC_AHP && c->ahp_scale != DC_AHP_SAATY9 && c->ahp_scale != DC_AHP_RATIO &&
        c->ahp_scale != DC_AHP_DIFF)
        return DC_EINVAL;
    if (c->method == DC_AHP && c->mode != DC_MODE_PLAIN) return DC_EINVAL;
    const int caps[5] = {c->host_cpu, c->host_ram, c->bw_host_edge, c->bw_edge_agg, c->bw_agg_core};
    for (int v : caps)
        if (v < 0 || v >= (1 << 22)) return DC_EINVAL;   // exact in FP32; fits the 22-bit path keys
    if (c->ncrit < 1 || c->ncrit > DC_MAX_CRIT) return DC_EINVAL;
    double ws = 0.0;
    for (int i = 0; i < c->ncrit; ++i) {
        if (c->crit[i] < DC_CRIT_CPU || c->crit[i] > DC_CRIT_HOPS) return DC_EINVAL;
        if (!(c->weight[i] > 0.f) || !std::isfinite(c->weight[i])) return DC_EINVAL;
        ws += c->weight[i];
    }
    if (std::fabs(ws - 1.0) > 1e-5) return DC_EINVAL;
    if (c->block != 0 && c->block != 64 && c->block != 256 && c->block != 512 && c->block != 1024) return DC_EINVAL;
    if (c->trace_stride < 0 || c->trace_cap < 0) return DC_EINVAL;
    if (c->grid < 0 || c->grid > 2) return DC_EINVAL;
    if (c->graph < 0 || c->graph > 2) return DC_EINVAL;
    if (c->grid_timeout_us < 0) return DC_EINVAL;
    if (c->routing < 0 || c->routing > 1) return DC_EINVAL;
    return DC_OK;
}

// Links of the path between servers u != v for candidate c, as global link
// ids (level * N + index); returns the count.
int host_path_links(const Topo &t, int u, int v, int c, int *out) {
    const int eu = u / t.h, ev = v / t.h, pu = u / t.hh, pv = v / t.hh;
    int a = 0, j = 0;
    if (pu == pv) a = c; else { a = c / t.h; j = c - a * t.h; }
    int nl = 0;
    out[nl++] = u;
    if (eu != ev) out[nl++] = t.N + eu * t.h + a;
    if (pu != pv) {
        out[nl++] = 2 * t.N + (pu * t.h + a) * t.h + j;
        out[nl++] = 2 * t.N + (pv * t.h + a) * t.h + j;
    }
    if (eu != ev) out[nl++] = t.N + ev * t.h + a;
    out[nl++] = v;
    return nl;
}

template <class K>
int set_lds(dc_ctx *ctx, K kernel, size_t bytes) {
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(bytes)));
    return DC_OK;
}

State state_of(dc_ctx *ctx, int inst) {
    int *s = ctx->d_state + (size_t)inst * 6 * ctx->N;
    const int N = ctx->N;
    return State{s, s + N, s + 2 * N, s + 3 * N, s + 4 * N, s + 5 * N};
}

Params base_params(dc_ctx *ctx, const DevBatch &b, int inst) {
    Params p{};
    p.t = ctx->t;
    p.st = state_of(ctx, inst);
    p.m = ctx->m;
    ahp_p1(ctx->m, p.p1);
    p.b = b.view;
    p.tr = Trace{ctx->d_tmeta, ctx->d_tscore, ctx->d_tcount, ctx->cfg.trace_stride, ctx->cfg.trace_cap};
    p.xs = ctx->d_xs + (size_t)inst * xs_rows(ctx->m.nc) * ctx->N;
    p.pc_cap = ctx->pc_plain;
    p.inst = inst;
    p.state_base = ctx->d_state;
    p.state_stride = 6LL * ctx->N;
    p.colpart = ctx->d_colpart;
    p.rowpart = ctx->d_rowpart;
    p.ysort = ctx->d_ysort;
    p.wsort = ctx->d_wsort;
    p.ti = ctx->ti; p.tj = ctx->tj; p.nI = ctx->nI; p.nJ = ctx->nJ;
    return p;
}

// Output region of a batch: host[Ct], code[Pt], failat[R] (all -1), then
// status[R] (1), then score[Ct], tsb[R], tse[R] (0; the stamps are int64).
int reset_outputs(dc_ctx *ctx, DevBatch &b) {
    const long long neg = (long long)b.Ct + b.Pt + b.R, all = (long long)b.out_ints;
    hipLaunchKernelGGL(k_reset_outputs, dim3((unsigned)std::min<long long>(2048, (all + 255) / 256)), dim3(256), 0,
                       ctx->stream, b.dmem + b.in_ints, neg, neg + b.R, all);
    HIPCHK(hipGetLastError());
    return DC_OK;
}

// n int32 of device memory for a batch, 16-byte aligned.
int batch_alloc(dc_ctx *ctx, size_t n, int **out) {
    n = align4(n);
    if (ctx->slab_end - ctx->slab_at < n) {
        const size_t slab = std::max<size_t>(n, (size_t)1 << 18);      // 1 MiB
        int *m = nullptr;
        HIPCHK(hipMalloc(&m, slab * sizeof(int)));
        ctx->slabs.push_back(m);
        ctx->slab_at = 0;
        ctx->slab_end = slab;
    }
    *out = ctx->slabs.back() + ctx->slab_at;
    ctx->slab_at += n;
    return DC_OK;
}

// The pinned buffer, at least n int32; what it held is lost when it grows.
int pinned_at_least(dc_ctx *ctx, size_t n) {
    if (ctx->pinned_ints >= n) return DC_OK;
    HIPCHK(hipStreamSynchronize(ctx->stream));      // a copy from it may be under way
    if (ctx->pinned) HIPCHK(hipHostFree(ctx->pinned));
    ctx->pinned = nullptr;
    ctx->pinned_ints = 0;
    const size_t want = std::max<size_t>(n + n / 2, 1 << 14);
    HIPCHK(hipHostMalloc(reinterpret_cast<void **>(&ctx->pinned), want * sizeof(int), 0));
    ctx->pinned_ints = want;
    return DC_OK;
}

// Turn the pending queue into one uploaded batch (requests grouped by
// instance, FCFS order kept within an instance).  The copy from the pinned
// buffer is under way on return; the caller waits for the stream before it
// returns to its own caller.
int upload_pending(dc_ctx *ctx) {
    const size_t R = ctx->pend_ids.size();
    if (R == 0) return DC_OK;
    auto B = std::make_unique<DevBatch>();
    DevBatch &b = *B;
    b.R = (int)R;
    b.I = ctx->I;
    std::vector<int> order(R);
    for (size_t r = 0; r < R; ++r) order[r] = (int)r;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int c) { return ctx->pend_inst[a] < ctx->pend_inst[c]; });
    b.coff.assign(1, 0);
    b.poff.assign(1, 0);
    b.iroff.assign(ctx->I + 1, 0);
    b.cuoff.assign(1, 0);
    for (int idx : order) {
        const Units &U = ctx->pend_units[idx];
        b.ids.push_back(ctx->pend_ids[idx]);
        b.inst.push_back(ctx->pend_inst[idx]);
        b.iroff[ctx->pend_inst[idx] + 1]++;
        const int pbase = (int)b.pj.size();
        for (int g = 0; g < U.nu(); ++g) {
            b.cpu.push_back(U.cpu[g]);
            b.ram.push_back(U.ram[g]);
            b.cmax.push_back(U.cmax[g]);
            b.rmax.push_back(U.rmax[g]);
            b.first.push_back(U.first[g]);
            b.poff.push_back(pbase + U.poff[g + 1]);
        }
        b.pj.insert(b.pj.end(), U.pj.begin(), U.pj.end());
        b.pbw.insert(b.pbw.end(), U.pbw.begin(), U.pbw.end());
        b.pbmax.insert(b.pbmax.end(), U.pbmax.begin(), U.pbmax.end());
        b.mem.push_back(std::move(ctx->pend_units[idx].mem));
        b.coff.push_back((int)b.cpu.size());
        b.cnt.push_back(U.n);
        b.unit_of.insert(b.unit_of.end(), U.unit_of.begin(), U.unit_of.end());
        b.cuoff.push_back((int)b.unit_of.size());
    }
    for (int i = 0; i < ctx->I; ++i) b.iroff[i + 1] += b.iroff[i];
    b.Ct = (int)b.cpu.size();
    b.Pt = (int)b.pj.size();
    // device layout: inputs coff, cpu, ram, poff, pj, pbw, iroff, rid, cmax,
    // rmax, pbmax; outputs host, code, failat, status, score, stamps, then
    // the allocations cpua, rama, pbwa
    size_t n_in = (size_t)(b.R + 1) + 2 * b.Ct + (b.Ct + 1) + 2 * (size_t)b.Pt + (b.I + 1) + b.R + 2 * b.Ct + b.Pt;
    n_in += n_in & 1;   // keeps the int64 stamps in the output region 8-byte aligned
    b.o_alloc = (size_t)b.Ct + b.Pt + b.R + b.R + b.Ct + 1 + 4 * (size_t)b.R;
    const size_t n_out = b.o_alloc + 2 * (size_t)b.Ct + b.Pt;
    b.in_ints = n_in;
    b.out_ints = n_out;
    int prc = pinned_at_least(ctx, n_in);
    if (prc || (prc = batch_alloc(ctx, n_in + n_out, &b.dmem))) return prc;
    int *img = ctx->pinned;
    size_t o = 0;
    auto put = [&](const std::vector<int> &v) { std::memcpy(img + o, v.data(), v.size() * sizeof(int)); o += v.size(); };
    const size_t o_coff = o; put(b.coff);
    const size_t o_cpu = o; put(b.cpu);
    const size_t o_ram = o; put(b.ram);
    const size_t o_poff = o; put(b.poff);
    const size_t o_pj = o; put(b.pj);
    const size_t o_pbw = o; put(b.pbw);
    const size_t o_iroff = o; put(b.iroff);
    std::vector<int> rid32(b.R);
    for (int r = 0; r < b.R; ++r) rid32[r] = (int)(b.ids[r] & 0x7fffffff);
    const size_t o_rid = o; put(rid32);
    const size_t o_cmax = o; put(b.cmax);
    const size_t o_rmax = o; put(b.rmax);
    const size_t o_pbmax = o; put(b.pbmax);
    if (o < n_in) img[o] = 0;
    HIPCHK(hipMemcpyAsync(b.dmem, img, n_in * sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    int *d = b.dmem;
    int *out = d + n_in;
    b.view.coff = d + o_coff;
    b.view.cpu = d + o_cpu;
    b.view.ram = d + o_ram;
    b.view.poff = d + o_poff;
    b.view.pj = d + o_pj;
    b.view.pbw = d + o_pbw;
    b.view.iroff = d + o_iroff;
    b.view.rid = d + o_rid;
    b.view.cmax = d + o_cmax;
    b.view.rmax = d + o_rmax;
    b.view.pbmax = d + o_pbmax;
    b.view.cpua = out + b.o_alloc;
    b.view.rama = out + b.o_alloc + b.Ct;
    b.view.pbwa = out + b.o_alloc + 2 * b.Ct;
    b.view.host = out;
    b.view.code = out + b.Ct;
    b.view.failat = out + b.Ct + b.Pt;
    b.view.status = out + b.Ct + b.Pt + b.R;
    b.view.score = reinterpret_cast<float *>(out + b.Ct + b.Pt + 2 * b.R);
    {
        size_t o_ts = (size_t)b.Ct + b.Pt + 2 * b.R + b.Ct;
        o_ts += o_ts & 1;   // n_in is even, so this makes the stamps 8-byte aligned
        b.view.tsb = reinterpret_cast<long long *>(out + o_ts);
        b.view.tse = b.view.tsb + b.R;
    }
    int rc = reset_outputs(ctx, b);
    if (rc) return rc;
    const int bi = (int)ctx->batches.size();
    for (int r = 0; r < b.R; ++r) ctx->loc[b.ids[r]] = ReqLoc{bi, r, false};
    ctx->batches.push_back(std::move(B));
    ctx->queued.push_back(bi);
    ctx->pend_ids.clear(); ctx->pend_inst.clear(); ctx->pend_units.clear();
    return DC_OK;
}

// The large AHP case: k = K with CPU, RAM, uplink, path bandwidth and hops
// (a cost), the list the CS = 5 kernels are compiled for.
bool specialised_ahp5(const dc_ctx *ctx, int K) {
    static const int crit[5] = {DC_CRIT_CPU, DC_CRIT_RAM, DC_CRIT_UPLINK, DC_CRIT_PATHBW, DC_CRIT_HOPS};
    if (ctx->t.k != K || ctx->m.method != DC_AHP || ctx->m.nc != 5) return false;
    for (int c = 0; c < 5; ++c)
        if (crit_of(ctx->m, c) != crit[c] || ctx->m.cost[c] != (c == 4)) return false;
    return true;
}

// Whether the context runs TOPSIS on the four default criteria (CPU, RAM,
// active, path bandwidth; all benefits), the list kernels are also compiled
// for; and on k = K fat-trees, for which some are compiled too.
bool default_criteria(const dc_ctx *ctx) {
    if (ctx->m.method != DC_TOPSIS || ctx->m.nc != 4) return false;
    for (int c = 0; c < 4; ++c)
        if (crit_of(ctx->m, c) != c || ctx->m.cost[c] != 0) return false;
    return true;
}
bool specialised(const dc_ctx *ctx, int K) { return ctx->t.k == K && default_criteria(ctx); }

// The kernel compiled for k = K, for the default criteria, or for any case.
template <class F>
F by_case(const dc_ctx *ctx, int K, F at_k, F at_list, F any) {
    return specialised(ctx, K) ? at_k : default_criteria(ctx) ? at_list : any;
}

// The cooperative and queue kernels compiled for k = 48 (the large data center
// of the serving form) on the default criteria, or for any case: a queue of
// 100 requests at k = 48 takes 16.8 ms, 19.1 with the sizes at run time.
constexpr int kGridK = 48;
const void *grid_step_kernel(const dc_ctx *ctx) {
    return reinterpret_cast<const void *>(by_case(ctx, kGridK, k_topsis_grid<kGridBlock, kGridK, 4>,
                                                  k_topsis_grid<kGridBlock, 0, 4>, k_topsis_grid<kGridBlock, 0, 0>));
}
const void *grid_serve_kernel(const dc_ctx *ctx) {
    return reinterpret_cast<const void *>(by_case(ctx, kGridK, k_serve_grid<kGridBlock, kGridK, 4>,
                                                  k_serve_grid<kGridBlock, 0, 4>, k_serve_grid<kGridBlock, 0, 0>));
}

// The AHP criteria kernel compiled for k = 32 (8,192 servers) on five criteria.
constexpr int kAhpK = 32;

template <int BS>
void launch_plain_step(dc_ctx *ctx, const Params &p) {
    if (ctx->use_grid) {
        Params pp = p;
        GridCtl g = ctx->grid;
        long long timeout = ctx->grid_timeout;
        void *args[] = {&pp, &g, &timeout};
        const hipError_t e = hipLaunchCooperativeKernel(grid_step_kernel(ctx), dim3(ctx->t.k), dim3(kGridBlock), args,
                                                        ctx->lds_grid, ctx->stream);
        if (e != hipSuccess && ctx->launch_err == hipSuccess) ctx->launch_err = e;
        ctx->last_launches += 1;
        return;
    }
    if (ctx->m.method == DC_TOPSIS) {
        hipLaunchKernelGGL((k_topsis_plain<BS>), dim3(1), dim3(BS), ctx->lds_plain, ctx->stream, p);
        ctx->last_launches += 1;
    } else {
        const int bx = (ctx->N + kAhpBlock - 1) / kAhpBlock;
        const int ncw = (ctx->N + BS - 1) / BS;        // criteria: BS servers a workgroup
        if (BS == 1024 && specialised_ahp5(ctx, kAhpK))
            hipLaunchKernelGGL((k_criteria_plain<1024, kAhpK, 5>), dim3(ncw), dim3(BS), ctx->lds_plain, ctx->stream,
                               p);
        else
            hipLaunchKernelGGL((k_criteria_plain<BS>), dim3(ncw), dim3(BS), ctx->lds_plain, ctx->stream, p);
        if (ctx->ahp_sorted) {
            Params q = p;
            q.nJ = 1;
            const dim3 gs(ctx->sort_runs, 1, ctx->m.nc), bs(kAhpSortBlock);
            hipLaunchKernelGGL(k_ahp_sort_runs, gs, bs, 0, ctx->stream, q, ctx->d_runs);
            if (ctx->sort_runs > 1) {
                hipLaunchKernelGGL(k_ahp_merge_runs, gs, bs, 0, ctx->stream, q, ctx->d_runs);
                ctx->last_launches += 1;
            }
            hipLaunchKernelGGL(k_ahp_sort_col, dim3(bx, 1, ctx->m.nc), dim3(kAhpBlock), 0, ctx->stream, q);
            hipLaunchKernelGGL(k_ahp_sort_row, dim3(bx, 1, ctx->m.nc), dim3(kAhpBlock), 0, ctx->stream, q);
            hipLaunchKernelGGL(k_ahp_pg, dim3(bx), dim3(kAhpBlock), 0, ctx->stream, q, nullptr, nullptr);
            hipLaunchKernelGGL((k_ahp_select<BS>), dim3(1), dim3(BS), ctx->lds_select, ctx->stream, q);
            ctx->last_launches += 6;
        } else if (ctx->ahp_large) {
            const AhpLarge &a = ctx->large;
            hipLaunchKernelGGL(k_ahp_count, dim3((ctx->N + kAhpQueueBlock - 1) / kAhpQueueBlock, ctx->m.nc),
                               dim3(kAhpQueueBlock), ctx->lds_count, ctx->stream, p, a);
            hipLaunchKernelGGL(k_ahp_rows, dim3(a.first[ctx->m.nc]), dim3(kRowWaves * kWave), 0, ctx->stream, p, a);
            hipLaunchKernelGGL(k_ahp_row_total, dim3(bx, ctx->m.nc), dim3(kAhpBlock), 0, ctx->stream, p, a);
            hipLaunchKernelGGL(k_ahp_pg, dim3(bx), dim3(kAhpBlock), 0, ctx->stream, p, a.lsum, a.didx);
            hipLaunchKernelGGL((k_ahp_select<BS>), dim3(1), dim3(BS), ctx->lds_select, ctx->stream, p);
            ctx->last_launches += 6;
        } else {
            hipLaunchKernelGGL(k_ahp_colsum, dim3(bx, ctx->nI, ctx->m.nc), dim3(kAhpBlock), 0, ctx->stream, p);
            hipLaunchKernelGGL(k_ahp_rowsum, dim3(bx, ctx->nJ, ctx->m.nc), dim3(kAhpBlock), 0, ctx->stream, p);
            hipLaunchKernelGGL(k_ahp_pg, dim3(bx), dim3(kAhpBlock), 0, ctx->stream, p, nullptr, nullptr);
            hipLaunchKernelGGL((k_ahp_select<BS>), dim3(1), dim3(BS), ctx->lds_select, ctx->stream, p);
            ctx->last_launches += 5;
        }
    }
}

int run_resident(dc_ctx *ctx, DevBatch &b);
int run_queue(dc_ctx *ctx, DevBatch &b, bool *ran);

int run_plain(dc_ctx *ctx, DevBatch &b) {
    if (ctx->plain_res && ctx->m.method == DC_TOPSIS && !ctx->use_grid) return run_resident(ctx, b);
    if (ctx->queue != dc_ctx::QUEUE_NONE) {
        bool ran = false;
        const int rc = run_queue(ctx, b, &ran);
        if (rc || ran) return rc;
    }
    ctx->launch_err = hipSuccess;
    for (int r = 0; r < b.R; ++r) {
        Params p = base_params(ctx, b, b.inst[r]);
        const int g0 = b.coff[r], n = b.coff[r + 1] - g0;
        for (int i = 0; i < n; ++i) {
            const int g = g0 + i;
            p.s = StepIn{r, i, n, g0, g, b.poff[g], b.poff[g + 1] - b.poff[g], b.cpu[g], b.ram[g], b.cmax[g], b.rmax[g]};
            for (int q = 0; q < p.s.P; ++q) {
                p.pj[q] = b.pj[p.s.p0 + q];
                p.pbw[q] = b.pbw[p.s.p0 + q];
                p.pbmax[q] = b.pbmax[p.s.p0 + q];
            }
            switch (ctx->plain_bs) {
            case 64: launch_plain_step<64>(ctx, p); break;
            case 256: launch_plain_step<256>(ctx, p); break;
            case 512: launch_plain_step<512>(ctx, p); break;
            default: launch_plain_step<1024>(ctx, p); break;
            }
        }
        ctx->last_steps += n;
        HIPCHK(ctx->launch_err);
    }
    HIPCHK(hipGetLastError());
    return DC_OK;
}

size_t batched_lds(const dc_ctx *ctx, int pc) {
    return resident_lds_bytes(pc, ctx->t.nsw, ctx->N, xs_rows(ctx->m.nc), kMaxPairs);
}

// The resident kernel compiled for k = 16 fat-trees scored on the four
// default criteria (the constants fold into the kernel), or for any case.
constexpr int kBatchedK = 16;
using ResidentFn = void (*)(Params);
template <int BS, int G, bool QUEUE>
ResidentFn resident_case(const dc_ctx *ctx) {
    return by_case<ResidentFn>(ctx, kBatchedK, k_topsis_resident<BS, G, kBatchedK, 4, QUEUE>,
                               k_topsis_resident<BS, G, 0, 4, QUEUE>, k_topsis_resident<BS, G, 0, 0, QUEUE>);
}

template <int BS, int G>
void launch_batched_k(dc_ctx *ctx, const Params &p, size_t lds, hipStream_t stream) {
    hipLaunchKernelGGL((resident_case<BS, G, false>(ctx)), dim3(ctx->I), dim3(BS), lds, stream, p);
}

template <int BS, int G>
int set_lds_batched(dc_ctx *ctx, size_t lds) {
    return set_lds(ctx, resident_case<BS, G, false>(ctx), lds);
}

// sh must be a built shape with 1 <= sh.pc <= ctx->pc_batched (callers check)
void launch_batched(dc_ctx *ctx, DevBatch &b, const Shape &sh, hipStream_t stream) {
    Params p = base_params(ctx, b, 0);
    p.pc_cap = sh.pc;
    p.xrows = xs_rows(ctx->m.nc);
    p.rq_pairs = kMaxPairs;
    const size_t lds = batched_lds(ctx, sh.pc);
    switch (sh.bs * 10 + sh.g) {
    case 2561: launch_batched_k<256, 1>(ctx, p, lds, stream); break;
    case 2562: launch_batched_k<256, 2>(ctx, p, lds, stream); break;
    case 2564: launch_batched_k<256, 4>(ctx, p, lds, stream); break;
    case 5121: launch_batched_k<512, 1>(ctx, p, lds, stream); break;
    case 5122: launch_batched_k<512, 2>(ctx, p, lds, stream); break;
    case 5124: launch_batched_k<512, 4>(ctx, p, lds, stream); break;
    case 10242: launch_batched_k<1024, 2>(ctx, p, lds, stream); break;
    default: launch_batched_k<1024, 1>(ctx, p, lds, stream); break;
    }
}

// Plain form with the state in LDS: the whole queue in one launch of the
// resident kernel, one workgroup per instance.  Its LDS is cut to the queue:
// the accumulator rows only where a container has more peers than a chunk of
// path tables, and as many of them and of the request's pairs as fit.
constexpr size_t kLdsMax = 159 * 1024;   // 160 KiB of LDS, 1 KiB left for static shared memory

struct Resident {
    int pc = 0, rows = 0, pairs = 0;
    size_t lds = 0;
};

Resident resident_layout(const dc_ctx *ctx, int max_peers, int max_pairs) {
    const int nsw = ctx->t.nsw, nc = ctx->m.nc, need = std::max(max_peers, 1);
    Resident L;
    auto fits = [&](int pc, int rows, int pairs) { return resident_lds_bytes(pc, nsw, ctx->N, rows, pairs) <= kLdsMax; };
    L.pairs = std::min(kMaxPairs, std::max(kMaxN, max_pairs));
    if (!fits(1, nc + 1, L.pairs)) L.pairs = kMaxN;
    L.rows = fits(need, nc + 1, L.pairs) || fits(need, nc + 1, kMaxN) ? nc + 1 : xs_rows(nc);
    if (!fits(L.rows == nc + 1 ? need : std::min(need, 4), L.rows, L.pairs)) L.pairs = kMaxN;
    for (L.pc = need; L.pc > 1 && !fits(L.pc, L.rows, L.pairs);) --L.pc;
    L.lds = resident_lds_bytes(L.pc, nsw, ctx->N, L.rows, L.pairs);
    return L;
}

// The resident kernel for a queue at BS threads: one server per thread where
// that covers them, otherwise several; at the automatic size the one
// compiled for k = 16.
template <int BS>
ResidentFn resident_fn(const dc_ctx *ctx) {
    if (BS == 1024 && ctx->N <= BS) return resident_case<BS, 1, true>(ctx);
    return default_criteria(ctx)
               ? (ctx->N <= BS ? k_topsis_resident<BS, 1, 0, 4, true> : k_topsis_resident<BS, host_group(BS), 0, 4, true>)
               : (ctx->N <= BS ? k_topsis_resident<BS, 1, 0, 0, true> : k_topsis_resident<BS, host_group(BS), 0, 0, true>);
}
ResidentFn resident_fn_at(const dc_ctx *ctx, int bs) {
    return bs == 64 ? resident_fn<64>(ctx) : bs == 256 ? resident_fn<256>(ctx)
         : bs == 512 ? resident_fn<512>(ctx) : resident_fn<1024>(ctx);
}

int run_resident(dc_ctx *ctx, DevBatch &b) {
    int max_pairs = 0, max_peers = 0;
    for (int r = 0; r < b.R; ++r) max_pairs = std::max(max_pairs, b.poff[b.coff[r + 1]] - b.poff[b.coff[r]]);
    for (int g = 0; g < b.Ct; ++g) max_peers = std::max(max_peers, b.poff[g + 1] - b.poff[g]);
    const Resident L = resident_layout(ctx, max_peers, max_pairs);
    Params p = base_params(ctx, b, 0);
    p.pc_cap = L.pc;
    p.xrows = L.rows;
    p.rq_pairs = L.pairs;
    hipLaunchKernelGGL(resident_fn_at(ctx, ctx->plain_bs), dim3(ctx->I), dim3(ctx->plain_bs), L.lds, ctx->stream, p);
    HIPCHK(hipGetLastError());
    ctx->last_launches += 1;
    ctx->last_steps += b.Ct;
    return DC_OK;
}

// Captures the batch's launch into a graph on a private stream (capture is
// not allowed on the legacy default stream a caller may have handed in).
int capture_batched(dc_ctx *ctx, DevBatch &b, const Shape &sh) {
    if (b.gexec) {
        HIPCHK(hipGraphExecDestroy(b.gexec));
        b.gexec = nullptr;
    }
    if (!ctx->cap_stream) HIPCHK(hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
    hipGraph_t g = nullptr;
    HIPCHK(hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeThreadLocal));
    launch_batched(ctx, b, sh, ctx->cap_stream);
    const hipError_t le = hipGetLastError();
    const hipError_t ce = hipStreamEndCapture(ctx->cap_stream, &g);
    HIPCHK(le);
    HIPCHK(ce);
    const hipError_t ie = hipGraphInstantiate(&b.gexec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    HIPCHK(ie);
    b.gshape = sh;
    return DC_OK;
}

int run_batched(dc_ctx *ctx, DevBatch &b, const Shape &sh) {
    if (ctx->cfg.graph == 1) {
        launch_batched(ctx, b, sh, ctx->stream);
    } else {
        if (!b.gexec || !(b.gshape == sh)) {
            const int rc = capture_batched(ctx, b, sh);
            if (rc) return rc;
        }
        HIPCHK(hipGraphLaunch(b.gexec, ctx->stream));
    }
    HIPCHK(hipGetLastError());
    ctx->last_launches += 1;
    ctx->last_steps += b.Ct;   // upper bound: containers queued (steps stop at a rejection)
    return DC_OK;
}

// Copies the outputs back through the pinned buffer: the servers, then
// everything after the route codes (failed_at, status, scores, timestamps).
// The route codes stay on the device; dc_get_paths fetches the few it needs.
// The results go, in request id order, to *dst, which moves past them, as far
// as `room` reaches, the others to ctx->ready.
int collect(dc_ctx *ctx, DevBatch &b, dc_result **dst, int64_t *room) {
    const int *dout = b.dmem + b.in_ints;
    const size_t tail0 = (size_t)b.Ct + b.Pt, tail = b.o_alloc - tail0;   // the allocations stay on the device
    const int prc = pinned_at_least(ctx, tail0 + tail);
    if (prc) return prc;
    int *out = ctx->pinned;
    // few route codes cost less than a second copy
    const bool whole = b.Pt <= 1 << 14;
    if (whole) {
        HIPCHK(hipMemcpyAsync(out, dout, b.o_alloc * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    } else {
        HIPCHK(hipMemcpyAsync(out, dout, (size_t)b.Ct * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK(hipMemcpyAsync(out + b.Ct, dout + tail0, tail * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    }
    HIPCHK(hipStreamSynchronize(ctx->stream));
    const int *t0 = out + (whole ? tail0 : b.Ct);      // output offset tail0 maps here
    b.host.assign(out, out + b.Ct);
    b.failat.assign(t0, t0 + b.R);
    b.status.assign(t0 + b.R, t0 + 2 * b.R);
    b.score.resize(b.Ct);
    std::memcpy(b.score.data(), t0 + 2 * b.R, sizeof(float) * b.Ct);
    b.tsb.resize(b.R);
    b.tse.resize(b.R);
    const long long *ts = b.view.tsb;
    const size_t o_ts = (size_t)(reinterpret_cast<const int *>(ts) - dout) - tail0;
    std::memcpy(b.tsb.data(), t0 + o_ts, sizeof(long long) * b.R);
    std::memcpy(b.tse.data(), t0 + o_ts + 2 * (size_t)b.R, sizeof(long long) * b.R);
    // results in request id order
    std::vector<int> order(b.R);
    for (int r = 0; r < b.R; ++r) order[r] = r;
    if (!std::is_sorted(b.ids.begin(), b.ids.end()))
        std::sort(order.begin(), order.end(), [&](int a, int c) { return b.ids[a] < b.ids[c]; });
    const size_t at = ctx->ready.size();
    const size_t direct = at ? 0 : (size_t)std::min<int64_t>(*room, (int64_t)order.size());
    ctx->ready.resize(at + order.size() - direct);
    dc_result *first = *dst;
    *dst += direct;
    *room -= (int64_t)direct;
    for (size_t k = 0; k < order.size(); ++k) {
        const int r = order[k];
        dc_result &res = k < direct ? first[k] : ctx->ready[at + k - direct];
        const int g0 = b.coff[r], c0 = b.cuoff[r];
        res.req_id = b.ids[r];
        res.instance = b.inst[r];
        res.status = b.status[r];
        res.n = b.cnt[r];
        const int nu = b.coff[r + 1] - g0;       // failat == nu: the links did not fit
        res.failed_at = b.status[r] ? -1 : (b.failat[r] < nu ? b.first[g0 + b.failat[r]] : b.cnt[r]);
        // a container gets its pod's server and score; a rejected request
        // places nothing (its attempt stays readable through dc_get_attempt)
        for (int i = 0; i < res.n; ++i) {
            const int g = g0 + b.unit_of[c0 + i];
            res.host[i] = res.status ? b.host[g] : -1;
            res.score[i] = b.score[g];
        }
        std::fill(res.host + res.n, res.host + DC_MAX_CONTAINERS, -1);
        std::fill(res.score + res.n, res.score + DC_MAX_CONTAINERS, 0.f);
    }
    return DC_OK;
}

// ---------------------------------------------------------------- cooperative step
int grid_alloc(dc_ctx *ctx, int G, size_t more = 0, unsigned long long **extra = nullptr) {
    // count, gen, err, round, join[2], done, reported, then 8-byte aligned:
    // kslot[2][G], rflag, rec[kRecWords][k], times, cmd, and `more` words
    const size_t own = 2 * (size_t)G + 1 + (size_t)ctx->t.k * kRecWords + 2 * kCmdRing + kCmdRing * kCmdWords;
    const size_t words = own + more;
    const size_t ints = 8 + 2 * words;
    HIPCHK(hipMalloc(&ctx->d_grid, ints * sizeof(int)));
    hipLaunchKernelGGL(k_fill_i32, dim3(more ? 64 : 16), dim3(256), 0, ctx->stream, ctx->d_grid, 0, (long long)ints);
    HIPCHK(hipGetLastError());
    int *p = ctx->d_grid;
    GridCtl &g = ctx->grid;
    g.count = reinterpret_cast<unsigned *>(p);
    g.gen = reinterpret_cast<unsigned *>(p + 1);
    g.err = p + 2;
    g.round = reinterpret_cast<unsigned *>(p + 3);
    g.join = reinterpret_cast<unsigned *>(p + 4);
    g.done = p + 6;
    g.reported = p + 7;
    g.kslot = reinterpret_cast<unsigned long long *>(p + 8);
    g.rflag = g.kslot + 2 * G;
    g.rec = g.rflag + 1;
    g.times = reinterpret_cast<long long *>(g.rec + (size_t)ctx->t.k * kRecWords);
    g.cmd = reinterpret_cast<unsigned long long *>(g.times + 2 * kCmdRing);
    g.wgs = G;
    g.pods = ctx->t.k;
    if (extra) *extra = g.kslot + own;
    return DC_OK;
}

int grid_init(dc_ctx *ctx) {
    const int G = ctx->t.k, h = ctx->t.h;
    if (h > kRecCapP - kRecCapE || G > kWave) return DC_EINVAL;
    const int rc = grid_alloc(ctx, G);
    if (rc) return rc;
    ctx->lds_grid = gsmem_bytes(h, ctx->t.hh, ctx->m.nc);
    const size_t serve_lds = align4(ctx->lds_grid / sizeof(int)) * sizeof(int) + req_lds_ints() * sizeof(int);
    if (serve_lds > 159 * 1024) return DC_EINVAL;
    if (hipFuncSetAttribute(grid_step_kernel(ctx), hipFuncAttributeMaxDynamicSharedMemorySize, (int)ctx->lds_grid) !=
            hipSuccess ||
        hipFuncSetAttribute(grid_serve_kernel(ctx), hipFuncAttributeMaxDynamicSharedMemorySize, (int)serve_lds) !=
            hipSuccess)
        return DC_EDEVICE;
    ctx->use_grid = true;
    return DC_OK;
}

// ---------------------------------------------------------------- queue kernels
using TopsisQueueFn = void (*)(Params, GridCtl, unsigned, long long, long long);
TopsisQueueFn topsis_queue_fn(const dc_ctx *ctx) {
    return by_case<TopsisQueueFn>(ctx, kGridK, k_topsis_queue<kGridBlock, kGridK, 4>, k_topsis_queue<kGridBlock, 0, 4>,
                                  k_topsis_queue<kGridBlock, 0, 0>);
}

using AhpQueueFn = void (*)(Params, GridCtl, AhpGrid, unsigned, long long, long long);
AhpQueueFn ahp_queue_fn(const dc_ctx *ctx) {
    return ahp_queue_block(ctx->N) == kAhpQueueBlock ? k_ahp_queue<kAhpQueueBlock> : k_ahp_queue<kAhpQueueBlock / 2>;
}

// Largest value criterion c can take: residuals stay within the capacities,
// path bandwidth within the server's uplink, hops within six per peer.
int crit_max(const dc_ctx *ctx, int c) {
    const dc_config &cfg = ctx->cfg;
    switch (crit_of(ctx->m, c)) {
    case CRIT_CPU: return cfg.host_cpu;
    case CRIT_RAM: return cfg.host_ram;
    case CRIT_ACTIVE: return 1;
    case CRIT_HOPS: return 6 * (kMaxN - 1);
    default: return cfg.bw_host_edge;
    }
}

// AHP on the 1-9 scale by distinct value, where the counts of a criterion's
// values fit one workgroup's LDS (capacities up to some 72,300) and a count
// 16 bits; otherwise the pairwise passes remain.
int large_init(dc_ctx *ctx) {
    const int N = ctx->N, nc = ctx->m.nc;
    if (ctx->m.scale != DC_AHP_SAATY9 || ctx->ahp_sorted || N >= 1 << 16) return DC_OK;
    AhpLarge &a = ctx->large;
    int vmax = 0;
    a.groups = (ctx->nJ + kRowWaves * kRowChunks - 1) / (kRowWaves * kRowChunks);
    for (int c = 0; c < nc; ++c) {
        a.vmax[c] = crit_max(ctx, c);
        vmax = std::max(vmax, a.vmax[c]);
        const int distinct = std::min(N, a.vmax[c] + 1);
        const int block = a.vmax[c] < kRowFew ? kRowBlockFew : kRowBlock;
        a.first[c + 1] = a.first[c] + (distinct + block - 1) / block * a.groups;
    }
    ctx->lds_count = large_count_lds(vmax);
    if (vmax >= 1 << 17 || ctx->lds_count > kLdsMax) return DC_OK;
    if (set_lds(ctx, k_ahp_count, ctx->lds_count)) return DC_EDEVICE;
    const size_t n = (size_t)nc * N;
    HIPCHK(hipMalloc(&ctx->d_large, n * (sizeof(double) + 3 * sizeof(int)) + kMaxCrit * sizeof(int)));
    a.lsum = static_cast<double *>(ctx->d_large);
    a.sinv = reinterpret_cast<float *>(a.lsum + n);
    a.didx = reinterpret_cast<int *>(a.sinv + n);
    a.dist = a.didx + n;
    a.count = a.dist + n;
    ctx->ahp_large = true;
    return DC_OK;
}

// Which plain contexts run their queue in one launch over several
// workgroups: one data center, left to the automatic choice (grid = 0 and no
// block size asked for).  TOPSIS where the state does not fit one workgroup
// (from k = 20 to 22 on): a step over one workgroup per pod.  On the default
// criteria that is always the faster form (40 requests of two containers at
// k = 22: 1.27 ms step by step, 0.96 so).  With other lists, which no kernel is
// compiled for, the exchanges between workgroups of a smaller data center cost
// more than one workgroup's step: the same requests on five criteria took 1.48
// ms step by step and 1.84 so at k = 24, 1.71 and 1.91 at k = 26, 1.93 and
// 1.83 at k = 28, so those take it from kQueueAnyK on.  AHP on the 1-9 scale
// up to 8,192 servers, where the position table of every criterion fits LDS
// beside the prefix sums.  A device (or a partition of one) that cannot hold
// all the workgroups at once keeps to one launch per step.
constexpr int kQueueAnyK = 28;
template <class F>
bool all_resident(F kernel, int block, size_t lds, int wgs) {
    int dev = 0, cus = 0, per = 0;
    return hipGetDevice(&dev) == hipSuccess &&
           hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void *>(kernel), block, lds) ==
               hipSuccess &&
           (long long)per * cus >= wgs;
}

int queue_init(dc_ctx *ctx) {
    const dc_config &cfg = ctx->cfg;
    if (cfg.mode != DC_MODE_PLAIN || ctx->I != 1 || cfg.grid != 0 || cfg.block != 0) return DC_OK;
    const int k = ctx->t.k, h = ctx->t.h, hh = ctx->t.hh, nc = ctx->m.nc;
    size_t words = 0;
    if (ctx->m.method == DC_TOPSIS) {
        if (ctx->plain_res || (k < kQueueAnyK && !default_criteria(ctx))) return DC_OK;
        ctx->queue_wgs = k;
        ctx->lds_queue = align4(gsmem_bytes(h, hh, nc) / sizeof(int)) * sizeof(int) + kQueueReqInts * sizeof(int);
        if (set_lds(ctx, topsis_queue_fn(ctx), ctx->lds_queue)) return DC_EDEVICE;
        if (!all_resident(topsis_queue_fn(ctx), kGridBlock, ctx->lds_queue, k)) return DC_OK;
        ctx->queue = dc_ctx::QUEUE_TOPSIS;
    } else {
        if (!ctx->ahp_sorted) return DC_OK;
        int vmax = 0;
        for (int c = 0; c < nc; ++c) {
            ctx->ahp.vmax[c] = crit_max(ctx, c);
            vmax = std::max(vmax, ctx->ahp.vmax[c]);
        }
        ctx->ahp.fbytes = ((vmax + 3) / 2 * 4 + 15) & ~15;
        ctx->lds_queue = ahp_queue_lds(h, hh, ctx->N, ctx->ahp.fbytes);
        if (vmax >= 1 << 17 || ctx->lds_queue > kLdsMax) return DC_OK;
        // a workgroup per pod, and enough of them that a slice of a
        // criterion's ranks is one row per thread
        const int bs = ahp_queue_block(ctx->N);
        ctx->queue_wgs = std::max(k, nc * ((ctx->N + bs - 1) / bs));
        if (ctx->queue_wgs > kWave) return DC_OK;
        if (set_lds(ctx, ahp_queue_fn(ctx), ctx->lds_queue)) return DC_EDEVICE;
        if (!all_resident(ahp_queue_fn(ctx), bs, ctx->lds_queue, ctx->queue_wgs)) return DC_OK;
        words = (size_t)nc * ctx->N;
        ctx->queue = dc_ctx::QUEUE_AHP;
    }
    if (cfg.grid_timeout_us > 0) ctx->patience = 100LL * cfg.grid_timeout_us;
    // the value, column and rank words of an AHP step behind the records
    unsigned long long *w = nullptr;
    const int rc = grid_alloc(ctx, ctx->queue_wgs, 3 * words, &w);
    ctx->ahp.xw = w;
    ctx->ahp.zw = w + words;
    ctx->ahp.lw = w + 2 * words;
    return rc;
}

// Runs a batch in one launch; *ran is false when its workgroups did not
// meet in time and nothing was done.  Once they have met, a wait inside is
// bounded by two seconds: far above any step, and only a fault reaches it.
int run_queue(dc_ctx *ctx, DevBatch &b, bool *ran) {
    constexpr long long kWait = 200000000LL;
    const Params p = base_params(ctx, b, 0);
    const unsigned epoch = ++ctx->epoch;
    if (ctx->queue == dc_ctx::QUEUE_TOPSIS)
        hipLaunchKernelGGL(topsis_queue_fn(ctx), dim3(ctx->queue_wgs), dim3(kGridBlock), ctx->lds_queue, ctx->stream, p,
                           ctx->grid, epoch, ctx->patience, kWait);
    else
        hipLaunchKernelGGL(ahp_queue_fn(ctx), dim3(ctx->queue_wgs), dim3(ahp_queue_block(ctx->N)), ctx->lds_queue,
                           ctx->stream, p, ctx->grid, ctx->ahp, epoch, ctx->patience, kWait);
    HIPCHK(hipGetLastError());
    // err, round, join[2] into the pinned buffer (any upload from it lies before
    // this copy on the stream)
    const int prc = pinned_at_least(ctx, 4);
    if (prc) return prc;
    const int *ctl = ctx->pinned;
    HIPCHK(hipMemcpyAsync(ctx->pinned, ctx->grid.err, 4 * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    if (ctl[0]) {
        ctx->poisoned = true;
        std::fprintf(stderr, "libdcsched: a wait inside a queue kernel timed out\n");
        return DC_EDEVICE;
    }
    *ran = static_cast<unsigned>(ctl[3]) == 2 * epoch;
    ctx->last_launches += 1;
    if (*ran) ctx->last_steps += b.Ct;
    return DC_OK;
}

// A cooperative step that timed out at a barrier poisons the context.
int grid_check(dc_ctx *ctx) {
    if (!ctx->use_grid) return DC_OK;
    int err = 0;
    HIPCHK(hipMemcpy(&err, ctx->grid.err, sizeof(int), hipMemcpyDeviceToHost));
    if (err) {
        ctx->poisoned = true;
        std::fprintf(stderr, "libdcsched: a cooperative step timed out at a grid barrier\n");
        return DC_EDEVICE;
    }
    return DC_OK;
}

// ---------------------------------------------------------------- serving form
int serve_init(dc_ctx *ctx) {
    auto sv = std::make_unique<Serve>();
    const size_t budget = ctx->cfg.mem_budget ? ctx->cfg.mem_budget : (size_t)256 << 20;
    sv->arena_ints = budget / sizeof(int);
    sv->stage_ints = slot_layout(kMaxN, kMaxPairs).in_end;
    const unsigned fl = hipHostMallocCoherent | hipHostMallocMapped;
    HIPCHK(hipHostMalloc(reinterpret_cast<void **>(&sv->cmds), sizeof(Cmd) * sv->cap, fl));
    HIPCHK(hipHostMalloc(reinterpret_cast<void **>(&sv->comps), sizeof(Comp) * sv->cap, fl));
    HIPCHK(hipHostMalloc(reinterpret_cast<void **>(&sv->ctrl), sizeof(int) * 4, fl));
    HIPCHK(hipHostMalloc(reinterpret_cast<void **>(&sv->staging), sizeof(int) * (size_t)sv->stage_ints * sv->cap, fl));
    std::memset(sv->cmds, 0, sizeof(Cmd) * sv->cap);
    std::memset(sv->comps, 0, sizeof(Comp) * sv->cap);
    std::memset(sv->ctrl, 0, sizeof(int) * 4);
    HIPCHK(hipMalloc(&sv->arena, sv->arena_ints * sizeof(int)));
    sv->free_list[0] = sv->arena_ints & ~size_t(3);
    HIPCHK(hipStreamCreateWithFlags(&sv->aux, hipStreamNonBlocking));
    sv->bs = ctx->N <= 256 ? 256 : 512;
    const size_t lds_max = kLdsMax;
    const size_t base = step_lds_bytes(0, ctx->t.nsw, req_lds_ints(), 0);
    sv->pc = (int)std::max<size_t>(1, std::min<size_t>(kMaxN, (lds_max - base) / (8 * (size_t)ctx->t.nsw)));
    sv->lds = step_lds_bytes(sv->pc, ctx->t.nsw, req_lds_ints(), 0);
    if (sv->lds > lds_max) return DC_EINVAL;
    if (set_lds(ctx, k_serve<256>, sv->lds) || set_lds(ctx, k_serve<512>, sv->lds)) return DC_EDEVICE;
    ctx->sv = std::move(sv);
    return DC_OK;
}

// (Re)launches the persistent kernel when commands wait and none runs.
int serve_ensure_running(dc_ctx *ctx) {
    Serve &sv = *ctx->sv;
    const int dev_pos = __atomic_load_n(sv.ctrl, __ATOMIC_ACQUIRE);
    if (dev_pos >= sv.host_pos) return DC_OK;
    if (sv.launched) {
        const hipError_t q = hipStreamQuery(ctx->stream);
        if (q == hipErrorNotReady) return DC_OK;      // still running: it will reach the command
        HIPCHK(q);
    }
    Params p{};
    p.t = ctx->t;
    p.st = state_of(ctx, 0);
    p.m = ctx->m;
    p.tr = Trace{nullptr, nullptr, nullptr, 0, 0};
    p.xs = ctx->d_xs;
    p.pc_cap = sv.pc;
    ServeArgs a{sv.cmds, sv.comps, sv.ctrl, sv.staging, sv.arena, sv.cap, sv.stage_ints, dev_pos, 0, sv.idle_ticks};
    __atomic_store_n(sv.ctrl + 1, 0, __ATOMIC_RELEASE);
    if (ctx->use_grid) {
        GridCtl g = ctx->grid;
        long long timeout = ctx->grid_timeout;
        void *args[] = {&p, &a, &g, &timeout};
        const size_t lds = align4(ctx->lds_grid / sizeof(int)) * sizeof(int) + req_lds_ints() * sizeof(int);
        // no command handed out before, and everything up to dev_pos reported
        hipLaunchKernelGGL(k_serve_reset, dim3(1), dim3(kWave), 0, ctx->stream, g, dev_pos);
        // the pods, and the two workgroups that talk to the host
        HIPCHK(hipLaunchCooperativeKernel(grid_serve_kernel(ctx), dim3(ctx->t.k + 2), dim3(kGridBlock), args, lds,
                                          ctx->stream));
    } else if (sv.bs == 256) {
        hipLaunchKernelGGL((k_serve<256>), dim3(1), dim3(256), sv.lds, ctx->stream, p, a);
    } else {
        hipLaunchKernelGGL((k_serve<512>), dim3(1), dim3(512), sv.lds, ctx->stream, p, a);
    }
    HIPCHK(hipGetLastError());
    sv.launched = true;
    return DC_OK;
}

// Publishes one command; the caller has checked ring space.
void serve_publish(Serve &sv, int type, int n, int P, size_t off, int rid) {
    Cmd &c = sv.cmds[sv.host_pos % sv.cap];
    c.type = type;
    c.n = n;
    c.npair = P;
    c.slot_off = (int)off;
    c.rid = rid;
    __atomic_store_n(&c.seq, (int)(sv.host_pos + 1), __ATOMIC_RELEASE);
    ++sv.host_pos;
}

int serve_poll(dc_ctx *ctx) {
    Serve &sv = *ctx->sv;
    if (ctx->use_grid && sv.launched && hipStreamQuery(ctx->stream) == hipSuccess) {
        int rc = grid_check(ctx);
        if (rc) return rc;
    }
    while (sv.comp_pos < sv.host_pos) {
        Comp &c = sv.comps[sv.comp_pos % sv.cap];
        if (__atomic_load_n(&c.seq, __ATOMIC_ACQUIRE) != (int)(sv.comp_pos + 1)) break;
        auto rit = sv.rid_to_id.find(c.rid);
        if (rit != sv.rid_to_id.end()) {
            const int64_t id = rit->second;
            ServeSlot &sl = sv.slots[id];
            if (c.type == CMD_SUBMIT) {
                sl.status = c.status;
                sl.hosts.resize(sl.nc);
                dc_result res;
                std::memset(&res, 0, sizeof res);
                res.req_id = id;
                res.instance = 0;
                res.status = c.status;
                res.n = sl.nc;
                res.failed_at = c.status ? -1 : (c.failat < sl.n ? sl.first[c.failat] : sl.nc);
                for (int i = 0; i < DC_MAX_CONTAINERS; ++i) res.host[i] = -1;
                for (int i = 0; i < sl.nc; ++i) {           // each container takes its pod's result
                    const int g = sl.unit_of[i];
                    sl.hosts[i] = c.host[g];
                    res.host[i] = c.status ? c.host[g] : -1;
                    res.score[i] = c.score[g];
                }
                ctx->ready.push_back(res);
                sv.service_us.emplace_back(id, (float)((c.t_decide - c.t_admit) / 100.0));
                if (!c.status) serve_free(sv, sl.off, sl.ints);   // rejected: nothing left to release
            } else {
                serve_free(sv, sl.off, sl.ints);                   // departure done
            }
        }
        ++sv.comp_pos;
    }
    return serve_ensure_running(ctx);
}

int serve_submit(dc_ctx *ctx, Units &U, int64_t *req_id) {
    Serve &sv = *ctx->sv;
    int rc = serve_poll(ctx);
    if (rc) return rc;
    const int n = U.nu();
    const std::vector<int> &poff = U.poff, &pj = U.pj, &pbw = U.pbw;
    const int *cpu = U.cpu.data(), *ram = U.ram.data();
    const int P = (int)pj.size();
    const SlotLayout L = slot_layout(n, P);
    if (sv.host_pos - sv.comp_pos >= sv.cap) return DC_EAGAIN;
    size_t off = 0;
    if (!serve_alloc(sv, (size_t)L.total, &off)) return DC_EAGAIN;
    const int64_t id = ctx->next_id++;
    const int rid = (int)(id & 0x7fffffff);
    int *stg = sv.staging + (size_t)(sv.host_pos % sv.cap) * sv.stage_ints;
    stg[L.coff] = 0;
    stg[L.coff + 1] = n;
    std::memcpy(stg + L.cpu, cpu, sizeof(int) * n);
    std::memcpy(stg + L.ram, ram, sizeof(int) * n);
    std::memcpy(stg + L.poff, poff.data(), sizeof(int) * (n + 1));
    std::memcpy(stg + L.cmax, U.cmax.data(), sizeof(int) * n);
    std::memcpy(stg + L.rmax, U.rmax.data(), sizeof(int) * n);
    if (P) {
        std::memcpy(stg + L.pj, pj.data(), sizeof(int) * P);
        std::memcpy(stg + L.pbw, pbw.data(), sizeof(int) * P);
        std::memcpy(stg + L.pbmax, U.pbmax.data(), sizeof(int) * P);
    }
    stg[L.rid] = rid;
    ServeSlot sl;
    sl.off = off;
    sl.ints = (size_t)L.total;
    sl.n = n;
    sl.P = P;
    sl.nc = U.n;
    sl.unit_of = std::move(U.unit_of);
    sl.first = std::move(U.first);
    sl.mem = std::move(U.mem);
    sv.slots[id] = std::move(sl);
    sv.rid_to_id[rid] = id;
    serve_publish(sv, CMD_SUBMIT, n, P, off, rid);
    if (req_id) *req_id = id;
    return serve_ensure_running(ctx);
}

int serve_release(dc_ctx *ctx, int64_t req_id) {
    Serve &sv = *ctx->sv;
    int rc = serve_poll(ctx);
    if (rc) return rc;
    auto it = sv.slots.find(req_id);
    if (it == sv.slots.end() || it->second.released) return DC_ENOENT;
    ServeSlot &sl = it->second;
    if (sl.status < 0) return DC_EAGAIN;          // not decided yet
    if (sl.status == 0) return DC_ENOENT;         // rejected: holds nothing
    if (sv.host_pos - sv.comp_pos >= sv.cap) return DC_EAGAIN;
    sl.released = true;
    serve_publish(sv, CMD_RELEASE, sl.n, sl.P, sl.off, (int)(req_id & 0x7fffffff));
    return serve_ensure_running(ctx);
}

// Stops the persistent kernel: publishes STOP and waits (bounded) for it.
int serve_stop(dc_ctx *ctx) {
    Serve &sv = *ctx->sv;
    if (!sv.launched) return DC_OK;
    const auto t0 = std::chrono::steady_clock::now();
    while (sv.host_pos - sv.comp_pos >= sv.cap) {
        int rc = serve_poll(ctx);
        if (rc) return rc;
        if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(60)) return DC_EDEVICE;
    }
    if (hipStreamQuery(ctx->stream) == hipErrorNotReady) serve_publish(sv, CMD_STOP, 0, 0, 0, -1);
    while (hipStreamQuery(ctx->stream) == hipErrorNotReady) {
        std::this_thread::sleep_for(std::chrono::microseconds(100));
        if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(60)) return DC_EDEVICE;
    }
    sv.launched = false;
    return DC_OK;
}

}  // namespace

namespace {

// A shape the current context can launch: a built (threads, servers per
// thread) pair and a peer chunk its LDS holds (batched form), or a plain
// workgroup size with its fixed grouping and chunk.
bool shape_ok(const dc_ctx *ctx, const Shape &sh) {
    if (ctx->cfg.mode == DC_MODE_BATCHED)
        return batched_shape_built(sh.bs, sh.g) && sh.pc >= 1 && sh.pc <= ctx->pc_batched;
    return (sh.bs == 64 || sh.bs == 256 || sh.bs == 512 || sh.bs == 1024) && sh.g == host_group(sh.bs) &&
           sh.pc == ctx->pc_plain;
}

// Cache key of a tuned shape: device architecture, form, method, servers,
// criteria.
std::string tune_key(const dc_ctx *ctx) {
    std::string arch = "unknown";
    int dev = 0;
    hipDeviceProp_t prop{};
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
        arch = prop.gcnArchName;
        const size_t colon = arch.find(':');
        if (colon != std::string::npos) arch.resize(colon);
    }
    const char *mode = ctx->cfg.mode == DC_MODE_BATCHED ? "batched" : "plain";
    const char *method = ctx->cfg.method == DC_AHP ? "ahp" : "topsis";
    return arch + "|" + mode + "|" + method + "|N=" + std::to_string(ctx->N) + "|C=" + std::to_string(ctx->m.nc);
}

// The cache is a text file of JSON objects, one per line:
// {"key": "...", "block": B, "host_group": G, "peer_chunk": P, "ms": T}
bool field_int(const std::string &line, const char *name, int *v) {
    const std::string pat = std::string("\"") + name + "\": ";
    const size_t at = line.find(pat);
    return at != std::string::npos && std::sscanf(line.c_str() + at + pat.size(), "%d", v) == 1;
}

std::string line_key(const std::string &line) {
    const std::string pat = "\"key\": \"";
    const size_t at = line.find(pat);
    if (at == std::string::npos) return std::string();
    const size_t end = line.find('"', at + pat.size());
    return end == std::string::npos ? std::string() : line.substr(at + pat.size(), end - at - pat.size());
}

bool cache_read(const char *path, const std::string &key, Shape *sh, float *ms) {
    std::ifstream in(path);
    std::string line;
    while (std::getline(in, line)) {
        if (line_key(line) != key) continue;
        int bs = 0, g = 0, pc = 0;
        if (!field_int(line, "block", &bs) || !field_int(line, "host_group", &g) || !field_int(line, "peer_chunk", &pc))
            return false;
        const size_t at = line.find("\"ms\": ");
        *ms = at == std::string::npos ? 0.f : std::strtof(line.c_str() + at + 6, nullptr);
        *sh = Shape{bs, g, pc};
        return true;
    }
    return false;
}

// Replaces (or adds) the key's line; written to a temporary file and renamed
// into place.  A cache that cannot be written is left as it was.
void cache_write(const char *path, const std::string &key, const Shape &sh, float ms) {
    std::vector<std::string> lines;
    {
        std::ifstream in(path);
        std::string line;
        while (std::getline(in, line))
            if (!line.empty() && line_key(line) != key) lines.push_back(line);
    }
    char buf[512];
    std::snprintf(buf, sizeof(buf), "{\"key\": \"%s\", \"block\": %d, \"host_group\": %d, \"peer_chunk\": %d, \"ms\": %.4f}",
                  key.c_str(), sh.bs, sh.g, sh.pc, ms);
    lines.push_back(buf);
    const std::string tmp = std::string(path) + ".tmp";
    {
        std::ofstream o(tmp, std::ios::trunc);
        if (!o) return;
        for (const auto &l : lines) o << l << "\n";
        if (!o) return;
    }
    (void)std::rename(tmp.c_str(), path);
}

}  // namespace

namespace {

// Which kernels score a set of tiles.
//   REG    a tile in the registers of one, four or sixteen wavefronts;
//   BIG    one workgroup per tile, reading it twice;
//   SPLIT  slices over several workgroups, statistics and scores in two
//          launches with partials in scratch.
enum { TILE_REG = 0, TILE_BIG = 1, TILE_SPLIT = 2 };
struct TilePath {
    int kind = TILE_BIG, C = 0, V = 0, W = 1, NW = 1;
    size_t scratch = 0;     // device bytes the launches need
    size_t refuse = 0;      // dc_topsis_tiles_noalloc: refused when above its static buffer
};

// Tiles past the registers: one workgroup each, in one launch without scratch,
// or the split.  One workgroup's time goes with the servers (a thread has C
// loads under way for each), the split's hardly.  One matrix not read before,
// with a mask and every score (us, one workgroup / split):
//   40,960 servers, C = 1 to 6:  34 / 40, 38 / 46, 43 / 48, 48 / 54, 55 / 60, 62 / 65
//   57,344, C = 1 to 4:          42 / 38, 47 / 46, 54 / 50, 62 / 55
//   4-byte loads, 12,289, C = 3 to 6: 41 / 47, 43 / 52, 48 / 57, 50 / 62
//   4-byte loads, 20,001, C = 3 to 6: 56 / 46, 60 / 52, 66 / 57, 70 / 61
// (from the caches the lines lie higher).  With 16-byte loads, tiles enough to
// fill the device are faster one workgroup each: 64 x 4 x 65,536 in 67 / 82.
// Past 1 MiB of criteria (512 KiB with 4-byte loads) always the split.
constexpr long long kBigTileInts = 1 << 18;
bool one_workgroup(int64_t T, int C, int N, bool vec) {
    if ((long long)C * N > (vec ? kBigTileInts : kBigTileInts / 2)) return false;
    return vec ? N <= 40960 || T >= 64 : N <= 14336;
}

// Fewest wavefronts (NW; 0: none) whose registers hold a tile: 4V servers per
// thread and criterion, V a power of two with C * V <= 16 (V <= 8).
struct TileRegs {
    int V, NW;
};
constexpr int tile_vmax(int C) { return C <= 2 ? 8 : C <= 4 ? 4 : 2; }
constexpr bool tile_built(int C, int V, int NW) {
    return V <= tile_vmax(C) && (NW == 1 || ((NW == 4 || NW == 16) && 4 * V > tile_vmax(C)));
}
constexpr TileRegs tile_regs(bool vec, int64_t T, int C, int N) {
    // with 4-byte loads half of that from two criteria on: 48 loads and more
    // a thread took longer than reading the tile twice (1,024 x 4 x 2,662: 48
    // against 32 us); several wavefronts are built from vmax / 4 < V on
    const int vcap = !vec && C > 1 && C <= 4 ? tile_vmax(C) / 2 : tile_vmax(C);
    const int vfirst = C <= 2 ? 4 : C <= 4 ? 2 : 1;
    for (int w = 1; w <= 16; w *= 4) {
        // 4-byte loads and few tiles, whose masks come a byte at a time: four
        // wavefronts from 257 servers on (64 tiles of 1 x 2,046 with masks 22 us
        // in one wavefront each, 11.4 in four; 4,096 of 1 x 510 0.6 times as fast)
        if (w == 1 && !vec && C <= 2 && N > 256 && T <= 512) continue;
        int v = w == 1 ? 1 : vfirst;
        while (v < vcap && 256 * v * w < N) v *= 2;
        if (256 * v * w >= N) return {v, w};
    }
    return {0, 0};
}

// Every choice is built: at each size where it changes, at both its sides.
constexpr bool tile_choices_built() {
    for (int C = 1; C <= DC_MAX_CRIT; ++C)
        for (int x = 0; x < 16; ++x)
            for (int n = 256 << (x / 2), k = 0; k < 4; ++k) {
                const TileRegs r = tile_regs(k & 1, k & 2 ? 512 : 513, C, n + (x & 1));
                if (r.NW && !tile_built(C, r.V, r.NW)) return false;
            }
    return true;
}
static_assert(tile_choices_built(), "a choice of tile_regs has no kernel");

int tiles_prepare(int64_t T, int32_t C, int32_t N, const int32_t *x, const uint8_t *feasible, const int32_t *cost,
                  const float *weight, float *scores, int32_t *best, float *best_score, TileArgs *a, TilePath *path) {
    if (T < 0 || T > 0x7fffffffLL || C < 1 || C > DC_MAX_CRIT || N < 1 || N > (1 << 20)) return DC_EINVAL;
    if (T == 0) return DC_OK;
    if (!x || !best || !weight) return DC_EINVAL;
    *a = TileArgs{};
    a->x = x;
    a->feas = feasible;
    a->scores = scores;
    a->best = best;
    a->best_score = best_score;
    a->C = C;
    a->N = N;
    for (int c = 0; c < C; ++c) {
        if (!(weight[c] > 0.f) || !std::isfinite(weight[c])) return DC_EINVAL;
        a->w[c] = weight[c];
        a->cost[c] = cost ? (cost[c] != 0) : 0;
    }
    auto al = [](const void *p, uintptr_t m) { return (reinterpret_cast<uintptr_t>(p) & (m - 1)) == 0; };
    const bool vec = N % 4 == 0 && al(x, 16) && (!scores || al(scores, 16)) && (!feasible || al(feasible, 4));
    path->C = C;
    path->W = vec ? 4 : 1;
    const TileRegs regs = tile_regs(vec, T, C, N);
    // the scratch of the two-launch split, which the calls of its range are
    // measured by against the static buffer whichever kernels they take
    const bool in_regs1 = vec && regs.NW == 1;
    const bool splits = !in_regs1 && N >= 2 * kSplitSlice && T <= kSplitMaxTiles;
    path->refuse = splits ? split_scratch_bytes(T, N, C) : 0;
    if (regs.NW) {
        path->kind = TILE_REG;
        path->V = regs.V;
        path->NW = regs.NW;
    } else if (one_workgroup(T, C, N, vec) || !splits) {
        path->kind = TILE_BIG;
    } else {
        path->kind = TILE_SPLIT;
        path->scratch = path->refuse;
    }
    return DC_OK;
}

template <int C, int V, int W>
int launch_tiles_reg(const TileArgs &a, int64_t T, int NW, hipStream_t st) {
    if (NW == 1) {
        // persistent grid: as many workgroups as fit on the device at once,
        // never more than needed for one wavefront per tile
        long long blocks = (T + kTileWaves - 1) / kTileWaves;
        if (blocks > 256) {
            int dev = 0, cus = 0, per = 0;
            if (hipGetDevice(&dev) != hipSuccess ||
                hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
                return DC_EDEVICE;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &per, reinterpret_cast<const void *>(k_topsis_tiles_reg<C, V, W, 1>), kTileBlock, 0) != hipSuccess ||
                per < 1)
                per = 1;
            blocks = std::min<long long>(blocks, (long long)per * cus);
        }
        hipLaunchKernelGGL((k_topsis_tiles_reg<C, V, W, 1>), dim3((unsigned)blocks), dim3(kTileBlock), 0, st, a,
                           (long long)T);
        return DC_OK;
    }
    // four wavefronts take what one cannot hold, sixteen what four cannot;
    // a workgroup per tile, within the launch's limit on threads
    const dim3 grid((unsigned)std::min<int64_t>(T, 1 << 20));
    if constexpr (tile_built(C, V, 4)) {
        if (NW == 4) hipLaunchKernelGGL((k_topsis_tiles_reg<C, V, W, 4>), grid, dim3(4 * kWave), 0, st, a, (long long)T);
        else hipLaunchKernelGGL((k_topsis_tiles_reg<C, V, W, 16>), grid, dim3(16 * kWave), 0, st, a, (long long)T);
        return DC_OK;
    }
    return DC_EDEVICE;      // not built, and not chosen (tile_choices_built)
}

template <int C, int W>
int launch_tiles_reg_v(const TileArgs &a, int64_t T, const TilePath &p, hipStream_t st) {
    switch (p.V) {
    case 1: return launch_tiles_reg<C, 1, W>(a, T, p.NW, st);
    case 2: return launch_tiles_reg<C, 2, W>(a, T, p.NW, st);
    case 4:
        if constexpr (C <= 4) return launch_tiles_reg<C, 4, W>(a, T, p.NW, st);
        break;
    case 8:
        if constexpr (C <= 2) return launch_tiles_reg<C, 8, W>(a, T, p.NW, st);
        break;
    }
    return DC_EDEVICE;      // not built, and not chosen (tile_choices_built)
}

template <int W>
int launch_tiles_reg_c(const TileArgs &a, int64_t T, const TilePath &p, hipStream_t st) {
    switch (p.C) {
    case 1: return launch_tiles_reg_v<1, W>(a, T, p, st);
    case 2: return launch_tiles_reg_v<2, W>(a, T, p, st);
    case 3: return launch_tiles_reg_v<3, W>(a, T, p, st);
    case 4: return launch_tiles_reg_v<4, W>(a, T, p, st);
    case 5: return launch_tiles_reg_v<5, W>(a, T, p, st);
    case 6: return launch_tiles_reg_v<6, W>(a, T, p, st);
    case 7: return launch_tiles_reg_v<7, W>(a, T, p, st);
    default: return launch_tiles_reg_v<8, W>(a, T, p, st);
    }
}

// work: path.scratch device bytes (unused when 0).
int tiles_launch(const TileArgs &a, int64_t T, const TilePath &path, void *work, hipStream_t st) {
    if (path.kind == TILE_REG) {
        const int rc = path.W == 4 ? launch_tiles_reg_c<4>(a, T, path, st) : launch_tiles_reg_c<1>(a, T, path, st);
        if (rc) return rc;
    } else if (path.kind == TILE_BIG) {
        const dim3 grid(static_cast<unsigned>(T)), block(kBigTileBlock);
        // (thousands of tiles of one criterion with 4-byte loads and masks, 1 x
        // 42,725: 1,024 threads took 1.15 times as long as 256)
        if (path.W == 4) hipLaunchKernelGGL(k_topsis_tiles_big<4>, grid, block, 0, st, a);
        else if (a.C == 1) hipLaunchKernelGGL((k_topsis_tiles_big<1, 256>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(k_topsis_tiles_big<1>, grid, block, 0, st, a);
    } else {
        const TileSplit sp = split_carve(work, T, a.N, a.C);
        const dim3 grid(static_cast<unsigned>(sp.S), static_cast<unsigned>(T));
        hipLaunchKernelGGL(k_tiles_split_stats, grid, dim3(kTileBlock), 0, st, a, sp);
        hipLaunchKernelGGL(k_tiles_split_score, grid, dim3(kTileBlock), 0, st, a, sp);
        hipLaunchKernelGGL(k_tiles_split_select, dim3(static_cast<unsigned>(T)), dim3(kWave), 0, st, a, sp);
    }
    if (hipGetLastError() != hipSuccess) return DC_EDEVICE;
    return DC_OK;
}

// Scratch of dc_topsis_tiles_noalloc: the split path's partials in a
// static device array, one copy per device, held until the process ends.
// Host code never passes the array's name to a kernel (on the host it is a
// stand-in, not a device address): the address comes from
// hipGetSymbolAddress, resolved once per device with that device current.
constexpr size_t kStaticScratchBytes = DC_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_addr[kMaxDevices] = {};

}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

// Device address of the current device's copy of `scratch`.
int static_scratch(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DC_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DC_EDEVICE;
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return DC_OK;
}

}  // namespace

extern "C" {

const char *dc_strerror(int code) {
    switch (code) {
    case DC_OK: return "ok";
    case DC_EINVAL: return "invalid argument";
    case DC_ENOMEM: return "out of memory";
    case DC_EAGAIN: return "memory budget full, retry later";
    case DC_ENOENT: return "unknown or not accepted request";
    case DC_EDEVICE: return "device error (context poisoned)";
    case DC_ESTATE: return "call not valid in this mode or state";
    case DC_ETOOBIG: return "needs more scratch than the static buffer holds";
    default: return "unknown error";
    }
}

int dc_create(const dc_config *cfg, dc_ctx **out) {
    if (!out) return DC_EINVAL;
    *out = nullptr;
    int rc = check_config(cfg);
    if (rc) return rc;
    const int k = cfg->k, h = k / 2, N = k * k * k / 4, I = cfg->n_instances;
    // background load must stay within capacity
    if (cfg->host_used)
        for (long long x = 0; x < (long long)I * 2 * N; ++x) {
            const int cap = ((x / N) % 2) ? cfg->host_ram : cfg->host_cpu;
            if (cfg->host_used[x] < 0 || cfg->host_used[x] > cap) return DC_EINVAL;
        }
    if (cfg->link_used)
        for (long long x = 0; x < (long long)I * 3 * N; ++x) {
            const int lvl = (int)((x / N) % 3);
            const int cap = lvl == 0 ? cfg->bw_host_edge : lvl == 1 ? cfg->bw_edge_agg : cfg->bw_agg_core;
            if (cfg->link_used[x] < 0 || cfg->link_used[x] > cap) return DC_EINVAL;
        }
    auto ctx = std::make_unique<dc_ctx>();
    ctx->cfg = *cfg;
    ctx->cfg.host_used = nullptr;
    ctx->cfg.link_used = nullptr;
    ctx->t = Topo{k, h, h * h, N, k * k / 2, 1.0f / h, 1.0f / (h * h), 1.0f / (k * k / 2)};
    ctx->N = N;
    ctx->I = I;
    ctx->m.method = cfg->method;
    ctx->m.scale = cfg->ahp_scale;
    ctx->m.nc = cfg->ncrit;
    ctx->m.route_end = cfg->routing;
    for (int c = 0; c < DC_MAX_CRIT; ++c) {
        ctx->m.codes |= c < cfg->ncrit ? static_cast<unsigned>(cfg->crit[c]) << (4 * c) : 0u;
        ctx->m.cost[c] = c < cfg->ncrit ? (cfg->crit_cost[c] != 0) : 0;
        ctx->m.w[c] = c < cfg->ncrit ? cfg->weight[c] : 0.f;
    }
    dc_ctx *c = ctx.get();
    if (cfg->stream) {
        c->stream = static_cast<hipStream_t>(cfg->stream);
    } else {
        if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess) return DC_EDEVICE;
        c->own_stream = true;
    }
    // initial state
    std::vector<int> init((size_t)I * 6 * N);
    for (int i = 0; i < I; ++i) {
        int *s = init.data() + (size_t)i * 6 * N;
        for (int u = 0; u < N; ++u) {
            s[u] = cfg->host_cpu - (cfg->host_used ? cfg->host_used[((size_t)i * 2) * N + u] : 0);
            s[N + u] = cfg->host_ram - (cfg->host_used ? cfg->host_used[((size_t)i * 2 + 1) * N + u] : 0);
            s[2 * N + u] = 0;
            const int caps[3] = {cfg->bw_host_edge, cfg->bw_edge_agg, cfg->bw_agg_core};
            for (int l = 0; l < 3; ++l)
                s[(3 + l) * N + u] = caps[l] - (cfg->link_used ? cfg->link_used[((size_t)i * 3 + l) * N + u] : 0);
        }
    }
    const size_t sbytes = init.size() * sizeof(int);
    if (hipMalloc(&c->d_state, sbytes) != hipSuccess || hipMalloc(&c->d_init, sbytes) != hipSuccess) {
        dc_destroy(ctx.release());
        return DC_ENOMEM;
    }
    if (hipMemcpy(c->d_init, init.data(), sbytes, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->d_state, init.data(), sbytes, hipMemcpyHostToDevice) != hipSuccess) {
        c->poisoned = true;
        dc_destroy(ctx.release());
        return DC_EDEVICE;
    }
    const int nc = cfg->ncrit;
    if (hipMalloc(&c->d_xs, (size_t)I * xs_rows(nc) * N * sizeof(int)) != hipSuccess) {
        dc_destroy(ctx.release());
        return DC_ENOMEM;
    }
    // launch shapes
    c->plain_bs = cfg->block ? cfg->block : (N <= 64 ? 64 : N <= 256 ? 256 : 1024);
    c->bshape.bs = cfg->block ? std::max(256, cfg->block) : 1024;
    c->bshape.g = c->bshape.bs >= 1024 ? 1 : host_group(c->bshape.bs);
    const size_t lds_max = kLdsMax;
    {
        // plain: state + scratch in LDS when they fit with at least 8 peer tables
        const size_t res_fixed = step_lds_bytes(0, c->t.nsw, (size_t)xs_rows(nc) * N, 6 * (size_t)N);
        const size_t per_peer = 8 * (size_t)c->t.nsw;
        c->plain_res = res_fixed + 8 * per_peer <= lds_max;
        if (c->plain_res) {
            c->pc_plain = (int)std::min<size_t>(kMaxN, (lds_max - res_fixed) / per_peer);
            c->lds_plain = step_lds_bytes(c->pc_plain, c->t.nsw, (size_t)xs_rows(nc) * N, 6 * (size_t)N);
        } else {
            c->pc_plain = (int)std::max<size_t>(1, std::min<size_t>(kMaxN, 64 * 1024 / per_peer));
            c->lds_plain = step_lds_bytes(c->pc_plain, c->t.nsw, 0, 0);
        }
    }
    c->lds_select = step_lds_bytes(0, c->t.nsw, 0, 0);
    if (cfg->mode == DC_MODE_BATCHED) {
        const size_t fixed = batched_lds(c, 0);
        if (fixed + 8 * (size_t)c->t.nsw > lds_max) { dc_destroy(ctx.release()); return DC_EINVAL; }
        c->pc_batched = (int)std::min<size_t>(kMaxN, (lds_max - fixed) / (8 * (size_t)c->t.nsw));
        c->bshape.pc = c->pc_batched;
        const size_t lb = batched_lds(c, c->pc_batched);
        if (set_lds_batched<256, 1>(c, lb) || set_lds_batched<256, 2>(c, lb) || set_lds_batched<256, 4>(c, lb) ||
            set_lds_batched<512, 1>(c, lb) || set_lds_batched<512, 2>(c, lb) || set_lds_batched<512, 4>(c, lb) ||
            set_lds_batched<1024, 1>(c, lb) || set_lds_batched<1024, 2>(c, lb)) {
            dc_destroy(ctx.release());
            return DC_EDEVICE;
        }
    }
    if (cfg->method == DC_TOPSIS && cfg->mode == DC_MODE_PLAIN &&
        (c->plain_res
             ? set_lds(c, resident_fn<64>(c), lds_max) || set_lds(c, resident_fn<256>(c), lds_max) ||
                   set_lds(c, resident_fn<512>(c), lds_max) || set_lds(c, resident_fn<1024>(c), lds_max)
             : set_lds(c, k_topsis_plain<64>, c->lds_plain) || set_lds(c, k_topsis_plain<256>, c->lds_plain) ||
                   set_lds(c, k_topsis_plain<512>, c->lds_plain) || set_lds(c, k_topsis_plain<1024>, c->lds_plain))) {
        dc_destroy(ctx.release());
        return DC_EDEVICE;
    }
    if (cfg->method == DC_AHP) {
        const int bx = (N + kAhpBlock - 1) / kAhpBlock;
        c->tj = std::min(N, 512);
        c->nJ = (N + c->tj - 1) / c->tj;
        c->nI = std::max(1, std::min(bx * 4, (2048 + bx * nc - 1) / (bx * nc)));
        c->ti = (N + c->nI - 1) / c->nI;
        c->nI = (N + c->ti - 1) / c->ti;
        // the 1-9 scale takes the sorted passes while a criterion's sorted
        // values and their prefix sums fit one workgroup's LDS
        c->ahp_sorted = cfg->ahp_scale == DC_AHP_SAATY9 && N <= kAhpSortMax;
        c->sort_runs = (N + kAhpSortBlock - 1) / kAhpSortBlock;
        const size_t colpart = (size_t)c->nI * sizeof(long long);
        if (hipMalloc(&c->d_colpart, (size_t)nc * N * colpart) != hipSuccess ||
            hipMalloc(&c->d_rowpart, (size_t)nc * c->nJ * N * sizeof(float)) != hipSuccess ||
            (c->ahp_sorted && (hipMalloc(&c->d_ysort, (size_t)nc * N * sizeof(int)) != hipSuccess ||
                               hipMalloc(&c->d_wsort, (size_t)nc * N * sizeof(double)) != hipSuccess ||
                               (c->sort_runs > 1 &&
                                hipMalloc(&c->d_runs, (size_t)nc * c->sort_runs * kAhpSortBlock * sizeof(int)) !=
                                    hipSuccess)))) {
            dc_destroy(ctx.release());
            return DC_ENOMEM;
        }
    }
    if (cfg->trace_stride > 0 && cfg->trace_cap > 0) {
        if (hipMalloc(&c->d_tmeta, (size_t)cfg->trace_cap * 4 * sizeof(int)) != hipSuccess ||
            hipMalloc(&c->d_tscore, (size_t)cfg->trace_cap * N * sizeof(float)) != hipSuccess ||
            hipMalloc(&c->d_tcount, (size_t)I * sizeof(int)) != hipSuccess) {
            dc_destroy(ctx.release());
            return DC_ENOMEM;
        }
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, c->stream, c->d_tcount, 0, (long long)I);
    }
    const bool grid_ok = cfg->method == DC_TOPSIS && cfg->mode != DC_MODE_BATCHED && I == 1;
    // automatic: the persistent serving kernel from k = 32 on; per-step
    // cooperative launches cost more to launch than they save, so the plain
    // form takes them only when asked (grid = 2)
    if (grid_ok && (cfg->grid == 2 || (cfg->grid == 0 && k >= 32 && cfg->mode == DC_MODE_SERVING))) {
        if (cfg->grid_timeout_us > 0) c->grid_timeout = 100LL * cfg->grid_timeout_us;   // 100 MHz clock
        const int grc = grid_init(c);
        if (grc) { dc_destroy(ctx.release()); return grc; }
    }
    if (cfg->method == DC_AHP && cfg->grid != 1) {
        const int lrc = large_init(c);
        if (lrc) { dc_destroy(ctx.release()); return lrc; }
    }
    if (const int qrc = queue_init(c)) { dc_destroy(ctx.release()); return qrc; }
    if (cfg->mode == DC_MODE_SERVING) {
        if (I != 1) { dc_destroy(ctx.release()); return DC_EINVAL; }
        const int src = serve_init(c);
        if (src) { dc_destroy(ctx.release()); return src; }
    }
    if (hipEventCreate(&c->ev0) != hipSuccess || hipEventCreate(&c->ev1) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        c->poisoned = true;
        dc_destroy(ctx.release());
        return DC_EDEVICE;
    }
    *out = ctx.release();
    return DC_OK;
}

int dc_submit_request_ranged(dc_ctx *ctx, int32_t instance, int32_t n, const int32_t *cpu_min,
                             const int32_t *cpu_max, const int32_t *ram_min, const int32_t *ram_max, int32_t m,
                             const int32_t *edges, const int32_t *bw_max, const int32_t *pod, int64_t *req_id) {
    if (!ctx) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (instance < 0 || instance >= ctx->I || n < 1 || n > DC_MAX_CONTAINERS || !cpu_min || !ram_min) return DC_EINVAL;
    if (m < 0 || m > n * (n - 1) / 2 || (m > 0 && !edges)) return DC_EINVAL;
    constexpr int kCap = 1 << 22;
    std::vector<char> seen((size_t)n * n, 0);
    for (int q = 0; q < m; ++q) {
        const int i = edges[3 * q], j = edges[3 * q + 1], bw = edges[3 * q + 2];
        const int bx = bw_max ? bw_max[q] : bw;
        if (i < 0 || j < 0 || i >= n || j >= n || i == j || bw <= 0 || bx < bw || bx > kCap) return DC_EINVAL;
        if (seen[(size_t)i * n + j]) return DC_EINVAL;
        seen[(size_t)i * n + j] = seen[(size_t)j * n + i] = 1;
    }
    for (int i = 0; i < n; ++i) {
        const int cx = cpu_max ? cpu_max[i] : cpu_min[i], rx = ram_max ? ram_max[i] : ram_min[i];
        if (cpu_min[i] < 0 || ram_min[i] < 0 || cx < cpu_min[i] || rx < ram_min[i] || cx > kCap || rx > kCap)
            return DC_EINVAL;
    }
    Units U;
    const int urc = build_units(n, cpu_min, cpu_max, ram_min, ram_max, m, edges, bw_max, pod, U);
    if (urc) return urc;
    if (ctx->sv) return serve_submit(ctx, U, req_id);
    ctx->pend_inst.push_back(instance);
    ctx->pend_units.push_back(std::move(U));
    const int64_t id = ctx->next_id++;
    ctx->pend_ids.push_back(id);
    if (req_id) *req_id = id;
    return DC_OK;
}

int dc_submit_request(dc_ctx *ctx, int32_t instance, int32_t n, const int32_t *cpu, const int32_t *ram,
                      int32_t m, const int32_t *edges, const int32_t *pod, int64_t *req_id) {
    return dc_submit_request_ranged(ctx, instance, n, cpu, nullptr, ram, nullptr, m, edges, nullptr, pod, req_id);
}

int dc_schedule(dc_ctx *ctx, int32_t max_results, dc_result *out, int32_t *n_out) {
    if (!ctx || max_results < 0 || (max_results > 0 && !out)) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    int rc = ctx->sv ? serve_poll(ctx) : upload_pending(ctx);
    if (rc) return rc;
    dc_result *dst = out;
    int64_t room = max_results;
    // results of earlier calls come first
    {
        const size_t k = std::min<size_t>((size_t)room, ctx->ready.size() - ctx->ready_head);
        if (k > 0) std::memcpy(dst, ctx->ready.data() + ctx->ready_head, sizeof(dc_result) * k);
        ctx->ready_head += k;
        dst += k;
        room -= (int64_t)k;
        if (ctx->ready_head == ctx->ready.size()) {
            ctx->ready.clear();
            ctx->ready_head = 0;
        }
    }
    if (!ctx->sv && !ctx->queued.empty()) {
        ctx->last_launches = 0;
        ctx->last_steps = 0;
        HIPCHK(hipEventRecord(ctx->ev0, ctx->stream));
        for (int bi : ctx->queued) {
            DevBatch &b = *ctx->batches[bi];
            rc = ctx->cfg.mode == DC_MODE_BATCHED ? run_batched(ctx, b, ctx->bshape) : run_plain(ctx, b);
            if (rc) return rc;
        }
        HIPCHK(hipEventRecord(ctx->ev1, ctx->stream));
        HIPCHK(hipGetLastError());
        for (int bi : ctx->queued) {
            rc = collect(ctx, *ctx->batches[bi], &dst, &room);
            if (rc) return rc;
        }
        rc = grid_check(ctx);
        if (rc) return rc;
        HIPCHK(hipEventElapsedTime(&ctx->last_ms, ctx->ev0, ctx->ev1));
        ctx->queued.clear();
    }
    if (n_out) *n_out = (int)(max_results - room);
    return DC_OK;
}

int dc_release(dc_ctx *ctx, int64_t req_id) {
    if (!ctx) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (ctx->sv) return serve_release(ctx, req_id);
    auto it = ctx->loc.find(req_id);
    if (it == ctx->loc.end() || it->second.released) return DC_ENOENT;
    DevBatch &b = *ctx->batches[it->second.batch];
    const int r = it->second.r;
    for (int bi : ctx->queued)
        if (bi == it->second.batch) return DC_ENOENT;   // not scheduled yet
    if ((int)b.status.size() <= r || b.status[r] != 1) return DC_ENOENT;
    Params p = base_params(ctx, b, b.inst[r]);
    p.s.r = r;
    hipLaunchKernelGGL((k_release<256>), dim3(1), dim3(256), 0, ctx->stream, p);
    HIPCHK(hipGetLastError());
    it->second.released = true;
    return DC_OK;
}

int dc_get_paths(dc_ctx *ctx, int64_t req_id, int32_t cap, int32_t *link_ids, int32_t *n) {
    if (!ctx || cap < 0 || (cap > 0 && !link_ids)) return DC_EINVAL;
    if (ctx->sv) {
        auto sit = ctx->sv->slots.find(req_id);
        if (sit == ctx->sv->slots.end() || sit->second.status != 1 || sit->second.released) return DC_ENOENT;
        const ServeSlot &sl = sit->second;
        std::vector<int> slot(sl.ints);
        HIPCHK(hipMemcpyAsync(slot.data(), ctx->sv->arena + sl.off, sl.ints * sizeof(int), hipMemcpyDeviceToHost,
                              ctx->sv->aux));
        HIPCHK(hipStreamSynchronize(ctx->sv->aux));
        const SlotLayout L = slot_layout(sl.n, sl.P);
        int q = 0;
        for (int g = 0; g < sl.n; ++g)
            for (int x = slot[L.poff + g]; x < slot[L.poff + g + 1]; ++x, ++q) {
                if (q >= cap) continue;
                int *dst = link_ids + 6 * (size_t)q;
                for (int l = 0; l < 6; ++l) dst[l] = -1;
                const int u = slot[L.host + g], v = slot[L.host + slot[L.pj + x]], c = slot[L.code + x];
                if (u != v && c >= 0) host_path_links(ctx->t, u, v, c, dst);
            }
        if (n) *n = q;
        return DC_OK;
    }
    auto it = ctx->loc.find(req_id);
    if (it == ctx->loc.end()) return DC_ENOENT;
    DevBatch &b = *ctx->batches[it->second.batch];
    const int r = it->second.r;
    if ((int)b.status.size() <= r || b.status[r] != 1) return DC_ENOENT;
    const int g0 = b.coff[r], g1 = b.coff[r + 1];
    const int x0 = b.poff[g0], nx = b.poff[g1] - x0;
    std::vector<int> code(std::max(nx, 1));
    if (nx > 0) {
        HIPCHK(hipMemcpyAsync(code.data(), b.view.code + x0, nx * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK(hipStreamSynchronize(ctx->stream));
    }
    int q = 0;
    for (int g = g0; g < g1; ++g)
        for (int x = b.poff[g]; x < b.poff[g + 1]; ++x, ++q) {
            if (q >= cap) continue;
            int *dst = link_ids + 6 * (size_t)q;
            for (int l = 0; l < 6; ++l) dst[l] = -1;
            const int u = b.host[g], v = b.host[g0 + b.pj[x]], c = code[x - x0];
            if (u != v && c >= 0) host_path_links(ctx->t, u, v, c, dst);
        }
    if (n) *n = q;
    return DC_OK;
}

int dc_get_alloc(dc_ctx *ctx, int64_t req_id, int32_t *cpu, int32_t *ram, int32_t *bw) {
    if (!ctx) return DC_EINVAL;
    if (ctx->sv) {
        auto sit = ctx->sv->slots.find(req_id);
        if (sit == ctx->sv->slots.end() || sit->second.status != 1 || sit->second.released) return DC_ENOENT;
        const ServeSlot &sl = sit->second;
        std::vector<int> slot(sl.ints);
        HIPCHK(hipMemcpyAsync(slot.data(), ctx->sv->arena + sl.off, sl.ints * sizeof(int), hipMemcpyDeviceToHost,
                              ctx->sv->aux));
        HIPCHK(hipStreamSynchronize(ctx->sv->aux));
        const SlotLayout L = slot_layout(sl.n, sl.P);
        members_alloc(sl.mem, sl.unit_of, sl.n, slot.data() + L.cpua, slot.data() + L.rama, slot.data() + L.pbwa,
                      cpu, ram, bw);
        return DC_OK;
    }
    auto it = ctx->loc.find(req_id);
    if (it == ctx->loc.end()) return DC_ENOENT;
    DevBatch &b = *ctx->batches[it->second.batch];
    const int r = it->second.r;
    if ((int)b.status.size() <= r || b.status[r] != 1) return DC_ENOENT;
    const int g0 = b.coff[r], nu = b.coff[r + 1] - g0;
    const int x0 = b.poff[g0], nx = b.poff[g0 + nu] - x0;
    std::vector<int> ua(2 * (size_t)nu + std::max(nx, 1));
    HIPCHK(hipMemcpyAsync(ua.data(), b.view.cpua + g0, nu * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipMemcpyAsync(ua.data() + nu, b.view.rama + g0, nu * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    if (nx > 0)
        HIPCHK(hipMemcpyAsync(ua.data() + 2 * nu, b.view.pbwa + x0, nx * sizeof(int), hipMemcpyDeviceToHost,
                              ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    const std::vector<int> uo(b.unit_of.begin() + b.cuoff[r], b.unit_of.begin() + b.cuoff[r + 1]);
    members_alloc(b.mem[r], uo, nu, ua.data(), ua.data() + nu, ua.data() + 2 * nu, cpu, ram, bw);
    return DC_OK;
}

int dc_get_attempt(dc_ctx *ctx, int64_t req_id, int32_t cap, int32_t *hosts, int32_t *n) {
    if (!ctx || cap < 0 || (cap > 0 && !hosts)) return DC_EINVAL;
    if (ctx->sv) {
        auto sit = ctx->sv->slots.find(req_id);
        if (sit == ctx->sv->slots.end() || sit->second.status < 0) return DC_ENOENT;
        const std::vector<int> &hv = sit->second.hosts;
        for (int i = 0; i < (int)hv.size() && i < cap; ++i) hosts[i] = hv[i];
        if (n) *n = (int)hv.size();
        return DC_OK;
    }
    auto it = ctx->loc.find(req_id);
    if (it == ctx->loc.end()) return DC_ENOENT;
    DevBatch &b = *ctx->batches[it->second.batch];
    const int r = it->second.r;
    if ((int)b.status.size() <= r) return DC_ENOENT;
    const int g0 = b.coff[r], c0 = b.cuoff[r], cnt = b.cnt[r];
    for (int i = 0; i < cnt && i < cap; ++i) hosts[i] = b.host[g0 + b.unit_of[c0 + i]];
    if (n) *n = cnt;
    return DC_OK;
}

int dc_get_latency(dc_ctx *ctx, int32_t cap, float *service_us, int32_t *n) {
    if (!ctx || cap < 0 || (cap > 0 && !service_us)) return DC_EINVAL;
    std::vector<std::pair<int64_t, float>> v;
    if (ctx->sv) v = ctx->sv->service_us;
    for (auto &B : ctx->batches) {
        const DevBatch &b = *B;
        for (int r = 0; r < (int)b.tse.size(); ++r)
            v.emplace_back(b.ids[r], (float)((b.tse[r] - b.tsb[r]) / 100.0));   // 100 MHz clock
    }
    std::sort(v.begin(), v.end());
    int k = 0;
    for (; k < (int)v.size() && k < cap; ++k) service_us[k] = v[k].second;
    if (n) *n = (int)v.size();
    return DC_OK;
}

int dc_get_state(dc_ctx *ctx, int32_t instance, int32_t *out) {
    if (!ctx || !out || instance < 0 || instance >= ctx->I) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    hipStream_t s = ctx->stream;
    if (ctx->sv) {
        int rc = serve_poll(ctx);
        if (rc) return rc;
        if (ctx->sv->comp_pos != ctx->sv->host_pos) return DC_EAGAIN;   // commands still in flight
        s = ctx->sv->aux;
    }
    HIPCHK(hipMemcpyAsync(out, ctx->d_state + (size_t)instance * 6 * ctx->N, 6 * (size_t)ctx->N * sizeof(int),
                          hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return DC_OK;
}

int dc_rewind(dc_ctx *ctx) {
    if (!ctx) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (ctx->sv) return DC_ESTATE;
    const bool fresh = !ctx->pend_ids.empty();
    int rc = upload_pending(ctx);
    if (rc) return rc;
    HIPCHK(hipMemcpyAsync(ctx->d_state, ctx->d_init, (size_t)ctx->I * 6 * ctx->N * sizeof(int),
                          hipMemcpyDeviceToDevice, ctx->stream));
    if (ctx->d_tcount)
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, ctx->stream, ctx->d_tcount, 0, (long long)ctx->I);
    ctx->queued.clear();
    for (size_t bi = 0; bi < ctx->batches.size(); ++bi) {
        rc = reset_outputs(ctx, *ctx->batches[bi]);
        if (rc) return rc;
        ctx->queued.push_back((int)bi);
        for (int64_t id : ctx->batches[bi]->ids) ctx->loc[id].released = false;
    }
    ctx->ready.clear();
    ctx->ready_head = 0;
    if (fresh) HIPCHK(hipStreamSynchronize(ctx->stream));
    return DC_OK;
}

int dc_get_trace(dc_ctx *ctx, int32_t cap, int32_t *meta, float *scores, int32_t *n) {
    if (!ctx || cap < 0) return DC_EINVAL;
    if (!ctx->d_tmeta) { if (n) *n = 0; return DC_OK; }
    std::vector<int> cnt(ctx->I);
    HIPCHK(hipMemcpyAsync(cnt.data(), ctx->d_tcount, ctx->I * sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    long long steps = 0;
    for (int v : cnt) steps = std::max<long long>(steps, v);
    int rec = (int)std::min<long long>(ctx->cfg.trace_cap, (steps + ctx->cfg.trace_stride - 1) / ctx->cfg.trace_stride);
    if (ctx->I > 1) rec = 0;   // per-instance counters share slots; recording is meant for one instance
    rec = std::min(rec, cap);
    if (rec > 0) {
        if (meta) HIPCHK(hipMemcpy(meta, ctx->d_tmeta, (size_t)rec * 4 * sizeof(int), hipMemcpyDeviceToHost));
        if (scores) HIPCHK(hipMemcpy(scores, ctx->d_tscore, (size_t)rec * ctx->N * sizeof(float), hipMemcpyDeviceToHost));
    }
    if (n) *n = rec;
    return DC_OK;
}

int dc_autotune(dc_ctx *ctx, int32_t *block) {
    dc_tune t{};
    const int rc = dc_autotune_cached(ctx, nullptr, &t);
    if (rc == DC_OK && block) *block = t.block;
    return rc;
}

int dc_autotune_cached(dc_ctx *ctx, const char *cache_path, dc_tune *out) {
    if (!ctx) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (ctx->cfg.mode == DC_MODE_SERVING) return DC_ESTATE;
    const bool batched = ctx->cfg.mode == DC_MODE_BATCHED;
    int rc = upload_pending(ctx);
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(ctx->stream));
    const std::string key = tune_key(ctx);
    if (cache_path && *cache_path) {
        Shape sh;
        float ms = 0.f;
        if (cache_read(cache_path, key, &sh, &ms) && shape_ok(ctx, sh)) {
            if (batched) ctx->bshape = sh; else ctx->plain_bs = sh.bs;
            if (out) *out = dc_tune{sh.bs, sh.g, sh.pc, 1, ms, 0};
            return DC_OK;
        }
    }
    if (ctx->queued.empty()) return DC_ESTATE;
    std::vector<Shape> cand;
    if (batched) {
        std::vector<int> pcs{ctx->pc_batched};
        for (int pc : {32, 16})
            if (pc < ctx->pc_batched) pcs.push_back(pc);
        for (const auto &x : kBatchedShapes)
            for (int pc : pcs) cand.push_back(Shape{x[0], x[1], pc});
    } else {
        for (int bs : {256, 512, 1024})
            if (bs == 256 || bs <= ctx->N) cand.push_back(Shape{bs, host_group(bs), ctx->pc_plain});   // no idle waves
    }
    // tuning runs record no trace and leave the state, the queue, the trace
    // counters and the current shape as they were
    struct Restore {
        dc_ctx *c;
        int stride, plain_bs, queue;
        bool use_grid;
        int *saved = nullptr;
        ~Restore() {
            c->cfg.trace_stride = stride;
            c->plain_bs = plain_bs;
            c->queue = queue;
            c->use_grid = use_grid;
            if (saved) (void)hipFree(saved);
        }
    } guard{ctx, ctx->cfg.trace_stride, ctx->plain_bs, ctx->queue, ctx->use_grid};
    ctx->cfg.trace_stride = 0;
    // the queue kernels and the cooperative step have their own block size:
    // what is tuned is the form that has one (and runs where a queue's
    // workgroups cannot meet), so that a cache entry always speaks of it
    ctx->queue = dc_ctx::QUEUE_NONE;
    ctx->use_grid = false;
    const size_t sbytes = (size_t)ctx->I * 6 * ctx->N * sizeof(int);
    HIPCHK(hipMalloc(&guard.saved, sbytes));
    HIPCHK(hipMemcpyAsync(guard.saved, ctx->d_state, sbytes, hipMemcpyDeviceToDevice, ctx->stream));
    float best_ms = 1e30f;
    Shape best = batched ? ctx->bshape : Shape{ctx->plain_bs, host_group(ctx->plain_bs), ctx->pc_plain};
    for (const Shape &sh : cand) {
        for (int rep = 0; rep < 2; ++rep) {   // first run warms up
            HIPCHK(hipMemcpyAsync(ctx->d_state, guard.saved, sbytes, hipMemcpyDeviceToDevice, ctx->stream));
            for (int bi : ctx->queued) if ((rc = reset_outputs(ctx, *ctx->batches[bi]))) return rc;
            HIPCHK(hipEventRecord(ctx->ev0, ctx->stream));
            ctx->plain_bs = sh.bs;
            for (int bi : ctx->queued) {
                if (batched) {
                    launch_batched(ctx, *ctx->batches[bi], sh, ctx->stream);   // timed eagerly
                    HIPCHK(hipGetLastError());
                } else if ((rc = run_plain(ctx, *ctx->batches[bi]))) {
                    return rc;
                }
            }
            HIPCHK(hipEventRecord(ctx->ev1, ctx->stream));
            HIPCHK(hipEventSynchronize(ctx->ev1));
            float ms = 0.f;
            HIPCHK(hipEventElapsedTime(&ms, ctx->ev0, ctx->ev1));
            if (rep == 1 && ms < best_ms) { best_ms = ms; best = sh; }
        }
    }
    HIPCHK(hipMemcpyAsync(ctx->d_state, guard.saved, sbytes, hipMemcpyDeviceToDevice, ctx->stream));
    for (int bi : ctx->queued) if ((rc = reset_outputs(ctx, *ctx->batches[bi]))) return rc;
    HIPCHK(hipStreamSynchronize(ctx->stream));
    if (batched) ctx->bshape = best; else guard.plain_bs = best.bs;
    if (cache_path && *cache_path) cache_write(cache_path, key, best, best_ms);
    if (out) *out = dc_tune{best.bs, best.g, best.pc, 0, best_ms, (int32_t)cand.size()};
    return DC_OK;
}

int dc_set_shape(dc_ctx *ctx, const dc_tune *shape) {
    if (!ctx || !shape) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (ctx->cfg.mode != DC_MODE_BATCHED) return DC_ESTATE;
    const Shape sh{shape->block, shape->host_group, shape->peer_chunk};
    if (!shape_ok(ctx, sh)) return DC_EINVAL;
    ctx->bshape = sh;
    return DC_OK;
}

int dc_get_shape(dc_ctx *ctx, dc_tune *shape) {
    if (!ctx || !shape) return DC_EINVAL;
    const Shape sh = ctx->cfg.mode == DC_MODE_BATCHED ? ctx->bshape
                                                       : Shape{ctx->plain_bs, host_group(ctx->plain_bs), ctx->pc_plain};
    *shape = dc_tune{sh.bs, sh.g, sh.pc, 0, 0.f, 0};
    return DC_OK;
}

int dc_pending(dc_ctx *ctx, int64_t *n) {
    if (!ctx || !n) return DC_EINVAL;
    if (ctx->poisoned) return DC_EDEVICE;
    if (ctx->sv) {
        int rc = serve_poll(ctx);
        if (rc) return rc;
        *n = ctx->sv->host_pos - ctx->sv->comp_pos;
    } else {
        int64_t q = (int64_t)ctx->pend_ids.size();
        for (int bi : ctx->queued) q += ctx->batches[bi]->R;
        *n = q;
    }
    return DC_OK;
}

int dc_topsis_tiles(int64_t T, int32_t C, int32_t N, const int32_t *x, const uint8_t *feasible,
                    const int32_t *cost, const float *weight, float *scores, int32_t *best, float *best_score,
                    void *stream) {
    TileArgs a{};
    TilePath path{};
    int rc = tiles_prepare(T, C, N, x, feasible, cost, weight, scores, best, best_score, &a, &path);
    if (rc || T == 0) return rc;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    if (!path.scratch) return tiles_launch(a, T, path, nullptr, st);
    // the split path's partials: stream-ordered allocation, freed behind the
    // launches (or, where the device has no stream-ordered allocator,
    // allocated and freed around a synchronised launch)
    void *scr = nullptr;
    const size_t bytes = path.scratch;
    if (hipMallocAsync(&scr, bytes, st) == hipSuccess) {
        rc = tiles_launch(a, T, path, scr, st);
        if (hipFreeAsync(scr, st) != hipSuccess) return DC_EDEVICE;
        return rc;
    }
    (void)hipGetLastError();
    if (hipMalloc(&scr, bytes) != hipSuccess) return DC_ENOMEM;
    rc = tiles_launch(a, T, path, scr, st);
    const bool done = hipStreamSynchronize(st) == hipSuccess;
    if (done) (void)hipFree(scr);      // left allocated if the device did not finish
    return done ? rc : DC_EDEVICE;
}

int dc_topsis_tiles_noalloc(int64_t T, int32_t C, int32_t N, const int32_t *x, const uint8_t *feasible,
                            const int32_t *cost, const float *weight, float *scores, int32_t *best,
                            float *best_score, void *stream) {
    TileArgs a{};
    TilePath path{};
    int rc = tiles_prepare(T, C, N, x, feasible, cost, weight, scores, best, best_score, &a, &path);
    if (rc) return rc;
    void *work = nullptr;
    if ((rc = static_scratch(&work))) return rc;     // the first call on a device resolves the address
    if (T == 0) return DC_OK;
    if (path.refuse > kStaticScratchBytes) return DC_ETOOBIG;
    return tiles_launch(a, T, path, work, static_cast<hipStream_t>(stream));
}

int dc_last_timing(dc_ctx *ctx, float *ms, int64_t *launches, int64_t *steps) {
    if (!ctx) return DC_EINVAL;
    if (ms) *ms = ctx->last_ms;
    if (launches) *launches = ctx->last_launches;
    if (steps) *steps = ctx->last_steps;
    return DC_OK;
}

void dc_destroy(dc_ctx *ctx) {
    if (!ctx) return;
    if (ctx->sv && !ctx->poisoned && serve_stop(ctx) != DC_OK) ctx->poisoned = true;
    // every kernel of this library ends on its own (bounded waits, idle exit),
    // so waiting for the streams is safe even on a poisoned context; memory is
    // freed only once nothing can still use it
    bool quiet = !ctx->stream || hipStreamSynchronize(ctx->stream) == hipSuccess;
    if (ctx->sv && ctx->sv->aux) quiet = hipStreamSynchronize(ctx->sv->aux) == hipSuccess && quiet;
    if (ctx->sv) {
        Serve &sv = *ctx->sv;
        if (quiet) {
            if (sv.cmds) (void)hipHostFree(sv.cmds);
            if (sv.comps) (void)hipHostFree(sv.comps);
            if (sv.ctrl) (void)hipHostFree(sv.ctrl);
            if (sv.staging) (void)hipHostFree(sv.staging);
            if (sv.arena) (void)hipFree(sv.arena);
        }
        if (sv.aux) (void)hipStreamDestroy(sv.aux);
    }
    if (quiet) {
        for (int *m : ctx->slabs) (void)hipFree(m);
        if (ctx->pinned) (void)hipHostFree(ctx->pinned);
        int *ptrs[] = {ctx->d_state, ctx->d_init, ctx->d_xs, ctx->d_colpart, ctx->d_tmeta, ctx->d_tcount, ctx->d_grid,
                       ctx->d_ysort, ctx->d_runs};
        for (int *p : ptrs)
            if (p) (void)hipFree(p);
        if (ctx->d_rowpart) (void)hipFree(ctx->d_rowpart);
        if (ctx->d_wsort) (void)hipFree(ctx->d_wsort);
        if (ctx->d_large) (void)hipFree(ctx->d_large);
        if (ctx->d_tscore) (void)hipFree(ctx->d_tscore);
    } else {
        std::fprintf(stderr, "libdcsched: the device did not finish this context's work; its memory is left allocated\n");
    }
    if (ctx->ev0) (void)hipEventDestroy(ctx->ev0);
    if (ctx->ev1) (void)hipEventDestroy(ctx->ev1);
    if (ctx->own_stream && ctx->stream) (void)hipStreamDestroy(ctx->stream);
    if (ctx->cap_stream) (void)hipStreamDestroy(ctx->cap_stream);
    delete ctx;
}

}  // extern "C"
