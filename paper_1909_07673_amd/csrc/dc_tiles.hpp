// TOPSIS scoring and selection (section V-C) over a batch of decision
// matrices that are already in device memory: T tiles of C integer criteria
// by N servers, criterion-major.  Per tile: exact column statistics (sum of
// squares, maximum, minimum), the closeness of every server with the same
// FP32 arithmetic as the fused container step, and the feasible server of
// highest closeness, lowest index on ties.  This is the scoring stage of the
// step on its own: a streaming pass bound by HBM bandwidth.
#pragma once
#include "dc_step.hpp"

namespace dcs {

struct TileArgs {
    const int *x;                 // [T][C][N] criteria, 0 <= value < 2^22
    const unsigned char *feas;    // [T][N] feasibility (nonzero = feasible), or null: all feasible
    float *scores;                // [T][N] closeness, or null
    int *best;                    // [T] chosen server, -1 when none is feasible
    float *best_score;            // [T] its closeness (0 when none), or null
    int C, N;
    float w[kMaxCrit];
    int cost[kMaxCrit];
};

constexpr int kTileBlock = 256;
constexpr int kTileWaves = kTileBlock / kWave;

// Block totals of per-thread column statistics; every thread receives them.
// The 64-bit sums of squares travel as three 17-bit chunks (as in the fused
// step), so no partial sum can overflow.
__device__ __forceinline__ void tile_stats(int C, unsigned long long *s2, int *mx, int *mn, int *wst) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        if (c >= C) break;
        const int c0 = wave_sum(static_cast<int>(s2[c] & 0x1ffffu));
        const int c1 = wave_sum(static_cast<int>((s2[c] >> 17) & 0x1ffffu));
        const int c2 = wave_sum(static_cast<int>(s2[c] >> 34));
        const int hi = wave_max(mx[c]), lo = wave_min(mn[c]);
        if (lane < 5) wst[(5 * c + lane) * kTileWaves + wid] = lane == 0 ? c0 : lane == 1 ? c1 : lane == 2 ? c2
                                                                 : lane == 3 ? hi : -lo;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        if (c >= C) break;
        int a0 = 0, a1 = 0, a2 = 0, hi = -kBig - 1, nlo = -kBig - 1;
#pragma unroll
        for (int x = 0; x < kTileWaves; ++x) {
            a0 += wst[(5 * c) * kTileWaves + x];
            a1 += wst[(5 * c + 1) * kTileWaves + x];
            a2 += wst[(5 * c + 2) * kTileWaves + x];
            hi = max(hi, wst[(5 * c + 3) * kTileWaves + x]);
            nlo = max(nlo, wst[(5 * c + 4) * kTileWaves + x]);
        }
        s2[c] = static_cast<unsigned long long>(static_cast<unsigned>(a0)) +
                (static_cast<unsigned long long>(static_cast<unsigned>(a1)) << 17) +
                (static_cast<unsigned long long>(static_cast<unsigned>(a2)) << 34);
        mx[c] = hi;
        mn[c] = -nlo;
    }
}

// Weighted normalisation folded into one factor per criterion, q = w^2 / S2,
// and the ideal / anti-ideal values (swapped for a cost criterion).
__device__ __forceinline__ void tile_factors(const TileArgs &a, const unsigned long long *s2, const int *mx,
                                             const int *mn, float *q, float *ap, float *am) {
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        q[c] = ap[c] = am[c] = 0.f;
        if (c >= a.C) continue;
        q[c] = s2[c] ? (a.w[c] * a.w[c]) / static_cast<float>(s2[c]) : 0.0f;
        ap[c] = static_cast<float>(a.cost[c] ? mn[c] : mx[c]);
        am[c] = static_cast<float>(a.cost[c] ? mx[c] : mn[c]);
    }
}

// A tile in registers: NW wavefronts hold all C criteria of one tile, each
// thread 4V servers of every criterion, so the tile crosses HBM exactly once
// (N <= 256 * V * NW, C * V <= 16: at most 64 registers of criteria).  With
// NW = 1 a workgroup's four wavefronts take a tile each, walking tiles with a
// grid stride, and every reduction is a wave DPP reduction, with no LDS and
// no barrier; otherwise the workgroup is one tile's.  W = 4: thread l takes
// the four-server groups l, l + 64 NW, ... with 16-byte loads (N % 4 == 0
// and aligned arrays); W = 1: servers l, l + 64 NW, ... with 4-byte loads,
// any N and alignment (each load still covers 256 consecutive bytes).
// Bound by HBM: 32,768 tiles of 4 x 1,024 in 89 us (one wavefront each, 6.0
// TB/s); 2,048 of 5 x 2,000 with every score in 23 us (four wavefronts,
// 4.4 TB/s), 71 us when a tile was read twice by 4-byte loads.
typedef int dcs_v4i __attribute__((ext_vector_type(4)));

// Block reduction of per-thread column statistics to the scoring factors:
// each wave reduces its own, then wave c the partials of criterion c, whose
// lane 0 turns them into q_c, A+_c and A-_c; every thread reads them after
// the barrier.  The per-wave 64-bit sums travel as three 20-bit chunks.
template <int NW, int C>
__device__ __forceinline__ void tile_factors_block(const TileArgs &a, int nc, const unsigned long long *s2,
                                                   const int *mx, const int *mn, float *q, float *ap, float *am) {
    __shared__ unsigned long long ps2[C][NW];
    __shared__ int pmx[C][NW], pmn[C][NW];
    __shared__ float f[3][C];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (c >= nc) break;
        const unsigned c0 = static_cast<unsigned>(wave_sum(static_cast<int>(s2[c] & 0x3ffffffu)));
        const unsigned c1 = static_cast<unsigned>(wave_sum(static_cast<int>((s2[c] >> 26) & 0x3ffffffu)));
        const unsigned c2 = static_cast<unsigned>(wave_sum(static_cast<int>(s2[c] >> 52)));
        const int hi = wave_max(mx[c]), lo = wave_min(mn[c]);
        if (lane == 0) {
            ps2[c][wid] = static_cast<unsigned long long>(c0) + (static_cast<unsigned long long>(c1) << 26) +
                          (static_cast<unsigned long long>(c2) << 52);
            pmx[c][wid] = hi;
            pmn[c][wid] = lo;
        }
    }
    __syncthreads();
    for (int c = wid; c < nc; c += NW) {
        const unsigned long long v = lane < NW ? ps2[c][lane] : 0ull;
        const int hi = wave_max(lane < NW ? pmx[c][lane] : -kBig - 1);
        const int lo = wave_min(lane < NW ? pmn[c][lane] : kBig);
        const unsigned c0 = static_cast<unsigned>(wave_sum(static_cast<int>(v & 0x3ffffffu)));
        const unsigned c1 = static_cast<unsigned>(wave_sum(static_cast<int>((v >> 26) & 0x3ffffffu)));
        const unsigned c2 = static_cast<unsigned>(wave_sum(static_cast<int>(v >> 52)));
        if (lane == 0) {
            const unsigned long long t = static_cast<unsigned long long>(c0) +
                                         (static_cast<unsigned long long>(c1) << 26) +
                                         (static_cast<unsigned long long>(c2) << 52);
            float w = 0.f;
            int cost = 0;
#pragma unroll
            for (int x = 0; x < C; ++x)
                if (x == c) { w = a.w[x]; cost = a.cost[x]; }
            f[0][c] = t ? (w * w) / static_cast<float>(t) : 0.0f;
            f[1][c] = static_cast<float>(cost ? lo : hi);
            f[2][c] = static_cast<float>(cost ? hi : lo);
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        q[c] = ap[c] = am[c] = 0.f;
        if (c >= C || c >= nc) continue;
        q[c] = f[0][c];
        ap[c] = f[1][c];
        am[c] = f[2][c];
    }
}

// Largest key over the block's NW wavefronts, in every lane of wave 0.
template <int NW>
__device__ __forceinline__ unsigned long long tile_block_max(unsigned long long kb) {
    __shared__ unsigned long long wkey[NW];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    unsigned hiw = wave_umax(static_cast<unsigned>(kb >> 32));
    unsigned low = wave_umax(static_cast<unsigned>(kb >> 32) == hiw ? static_cast<unsigned>(kb) : 0u);
    if (NW > 1) {
        if (lane == 0) wkey[wid] = (static_cast<unsigned long long>(hiw) << 32) | low;
        __syncthreads();
        if (wid == 0) {
            const unsigned long long k = lane < NW ? wkey[lane] : 0ull;
            hiw = wave_umax(static_cast<unsigned>(k >> 32));
            low = wave_umax(static_cast<unsigned>(k >> 32) == hiw ? static_cast<unsigned>(k) : 0u);
        }
    }
    return (static_cast<unsigned long long>(hiw) << 32) | low;
}

__device__ __forceinline__ void tile_write_best(const TileArgs &a, long long t, unsigned long long best) {
    a.best[t] = best ? static_cast<int>(~static_cast<unsigned>(best)) : -1;
    if (a.best_score) a.best_score[t] = best ? __uint_as_float(static_cast<unsigned>(best >> 32) - 1u) : 0.f;
}

template <int C, int V, int W, int NW>
__global__ __launch_bounds__(NW == 1 ? kTileBlock : NW *kWave) void k_topsis_tiles_reg(TileArgs a, long long T) {
    constexpr int E = 4 * V, L = NW * kWave, TW = NW == 1 ? kTileWaves : 1;
    const int l = NW == 1 ? threadIdx.x & (kWave - 1) : threadIdx.x;
    const int N = a.N;
    const size_t tile = static_cast<size_t>(C) * N;
    const long long step = static_cast<long long>(gridDim.x) * TW;
    for (long long t = static_cast<long long>(blockIdx.x) * TW + (NW == 1 ? threadIdx.x / kWave : 0); t < T;
         t += step) {
        const int *x = a.x + t * tile;
        // element e of thread l is server u(e)
        auto server = [&](int e) { return W == 4 ? 4 * ((e >> 2) * L + l) + (e & 3) : e * L + l; };
        int v[C][E];
#pragma unroll
        for (int e = 0; e < E; e += W) {
            const int u = server(e);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (W == 4) {
                    dcs_v4i r = {0, 0, 0, 0};
                    if (u < N)
                        r = __builtin_nontemporal_load(
                            reinterpret_cast<const dcs_v4i *>(x + static_cast<size_t>(c) * N + u));
                    v[c][e] = r.x; v[c][e + W / 4] = r.y; v[c][e + W / 2] = r.z; v[c][e + W - 1] = r.w;
                } else {
                    v[c][e] = u < N ? __builtin_nontemporal_load(x + static_cast<size_t>(c) * N + u) : 0;
                }
            }
        }
        // exact column statistics: per-thread 64-bit sums of squares (values
        // below 2^22, at most 4V <= 64 of them, so below 2^50)
        unsigned long long s2[kMaxCrit];
        int mx[kMaxCrit], mn[kMaxCrit];
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) { s2[c] = 0; mx[c] = -kBig - 1; mn[c] = kBig; }
#pragma unroll
        for (int e = 0; e < E; e += W) {
            if (server(e) >= N) break;             // servers ascend with e
#pragma unroll
            for (int c = 0; c < C; ++c) {
                int hi = v[c][e], lo = v[c][e];
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    const unsigned b = v[c][e + j];
                    s2[c] += static_cast<unsigned long long>(b) * b;
                    hi = max(hi, v[c][e + j]);
                    lo = min(lo, v[c][e + j]);
                }
                mx[c] = max(mx[c], hi);
                mn[c] = min(mn[c], lo);
            }
        }
        float q[kMaxCrit], ap[kMaxCrit], am[kMaxCrit];
        if (NW == 1) {
            // reduced as a low 26-bit chunk (64 lanes sum below 2^32) and the rest
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const unsigned lo = static_cast<unsigned>(wave_sum(static_cast<int>(s2[c] & 0x3ffffffu)));
                const unsigned hi = static_cast<unsigned>(wave_sum(static_cast<int>(s2[c] >> 26)));
                s2[c] = static_cast<unsigned long long>(lo) + (static_cast<unsigned long long>(hi) << 26);
                mx[c] = wave_max(mx[c]);
                mn[c] = wave_min(mn[c]);
            }
            tile_factors(a, s2, mx, mn, q, ap, am);
        } else {
            tile_factors_block<NW, C>(a, C, s2, mx, mn, q, ap, am);
        }
        unsigned long long kb = 0;
#pragma unroll
        for (int e = 0; e < E; e += W) {
            const int u = server(e);
            if (u >= N) break;
            unsigned fm = 0x01010101u;
            if (a.feas) {
                const unsigned char *fp = a.feas + static_cast<size_t>(t) * N + u;
                fm = W == 4 ? *reinterpret_cast<const unsigned *>(fp) : *fp;
            }
            float sc[W];
#pragma unroll
            for (int j = 0; j < W; ++j) {
                sc[j] = topsis_close(C, [&](int c) { return v[c < C ? c : 0][e + j]; }, q, ap, am);
                if ((fm >> (8 * j)) & 0xffu) {
                    const unsigned long long k = score_key(sc[j], u + j);
                    kb = k > kb ? k : kb;
                }
            }
            if (a.scores) {
                float *o = a.scores + static_cast<size_t>(t) * N + u;
                if (W == 4) *reinterpret_cast<float4 *>(o) = make_float4(sc[0], sc[W / 4], sc[W / 2], sc[W - 1]);
                else *o = sc[0];
            }
        }
        kb = tile_block_max<NW>(kb);
        if (l == 0) tile_write_best(a, t, kb);
        if (NW > 1) __syncthreads();               // LDS of the reductions is written again at the next tile
    }
}

// Tiles too large for the registers: one workgroup of 1,024 threads (256 where a
// server is one 4-byte load, dc_lib.hip) per tile,
// which reads the tile for its statistics and again, from the caches, for
// the scores.  A single tile takes one compute unit's cache bandwidth (at
// most 1 MiB, dc_lib.hip), yet one launch without scratch ends sooner than
// several workgroups would behind an allocation and a second launch.
constexpr int kBigTileBlock = 1024;

template <int W, int BS = kBigTileBlock>
__global__ __launch_bounds__(BS) void k_topsis_tiles_big(TileArgs a) {
    constexpr int NW = BS / kWave;
    const int t = blockIdx.x, N = a.N, C = a.C;
    const int *x = a.x + static_cast<size_t>(t) * C * N;
    unsigned long long s2[kMaxCrit];
    int mx[kMaxCrit], mn[kMaxCrit];
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) { s2[c] = 0; mx[c] = -kBig - 1; mn[c] = kBig; }
    auto load = [&](int c, int u, int *e) {
        const int *g = x + static_cast<size_t>(c) * N + u;
        if (W == 4) {
            const int4 r = *reinterpret_cast<const int4 *>(g);
            e[0] = r.x; e[W / 4] = r.y; e[W / 2] = r.z; e[W - 1] = r.w;
        } else {
            e[0] = *g;
        }
    };
#pragma unroll 2
    for (int u = W * threadIdx.x; u < N; u += W * BS) {
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) {
            if (c >= C) break;
            int e[W];
            load(c, u, e);
#pragma unroll
            for (int j = 0; j < W; ++j) {
                const unsigned b = e[j];
                s2[c] += static_cast<unsigned long long>(b) * b;
                mx[c] = max(mx[c], e[j]);
                mn[c] = min(mn[c], e[j]);
            }
        }
    }
    float q[kMaxCrit], ap[kMaxCrit], am[kMaxCrit];
    tile_factors_block<NW, kMaxCrit>(a, C, s2, mx, mn, q, ap, am);
    unsigned long long kb = 0;
    for (int u = W * threadIdx.x; u < N; u += W * BS) {
        int e[kMaxCrit][W];
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) {
            if (c < C) {
                load(c, u, e[c]);
            } else {
#pragma unroll
                for (int j = 0; j < W; ++j) e[c][j] = 0;
            }
        }
        unsigned fm = 0x01010101u;
        if (a.feas) {
            const unsigned char *fp = a.feas + static_cast<size_t>(t) * N + u;
            fm = W == 4 ? *reinterpret_cast<const unsigned *>(fp) : *fp;
        }
        float sc[W];
#pragma unroll
        for (int j = 0; j < W; ++j) {
            sc[j] = topsis_close(C, [&](int c) { return e[c][j]; }, q, ap, am);
            if ((fm >> (8 * j)) & 0xffu) {
                const unsigned long long k = score_key(sc[j], u + j);
                kb = k > kb ? k : kb;
            }
        }
        if (a.scores) {
            float *o = a.scores + static_cast<size_t>(t) * N + u;
            if (W == 4) *reinterpret_cast<float4 *>(o) = make_float4(sc[0], sc[W / 4], sc[W / 2], sc[W - 1]);
            else *o = sc[0];
        }
    }
    kb = tile_block_max<NW>(kb);
    if (threadIdx.x == 0) tile_write_best(a, t, kb);
}

// ---------------------------------------------------------------- large tiles
// A few tiles of many servers (a large data center's matrix) would leave
// most of the device idle at one workgroup per tile, so each tile is split
// into slices of kSplitSlice servers, one workgroup each, and the
// reductions go through partials in scratch memory:
//   1. per slice, the exact column statistics -> sp.s2, sp.mx, sp.mn;
//   2. per slice, the tile's totals from all slices (in slice order), the
//      closeness of the slice's servers and the slice's best key -> sp.key;
//   3. per tile, the best key over its slices.
// The totals are exact integers, so the scores are bit-identical to the
// other paths.
constexpr int kSplitSlice = 2048;
constexpr long long kSplitMaxTiles = 1024;   // more tiles fill the device at one workgroup each

struct TileSplit {
    unsigned long long *s2;   // [T][S][C] slice sums of squares
    int *mx, *mn;             // [T][S][C] slice maxima / minima
    unsigned long long *key;  // [T][S] slice best keys
    int S;                    // slices per tile
};

// Scratch bytes of the split path for T tiles of N servers and C criteria
// (each region 256-byte aligned).
__host__ __device__ inline size_t split_scratch_bytes(long long T, int N, int C) {
    const long long S = (N + kSplitSlice - 1) / kSplitSlice;
    auto al = [](long long b) { return static_cast<size_t>((b + 255) & ~255LL); };
    return al(T * S * C * 8) + 2 * al(T * S * C * 4) + al(T * S * 8);
}

__host__ __device__ inline TileSplit split_carve(void *base, long long T, int N, int C) {
    const long long S = (N + kSplitSlice - 1) / kSplitSlice;
    auto al = [](long long b) { return static_cast<size_t>((b + 255) & ~255LL); };
    char *p = static_cast<char *>(base);
    TileSplit sp;
    sp.S = static_cast<int>(S);
    sp.s2 = reinterpret_cast<unsigned long long *>(p); p += al(T * S * C * 8);
    sp.mx = reinterpret_cast<int *>(p); p += al(T * S * C * 4);
    sp.mn = reinterpret_cast<int *>(p); p += al(T * S * C * 4);
    sp.key = reinterpret_cast<unsigned long long *>(p);
    return sp;
}

// grid (S, T): column statistics of slice blockIdx.x of tile blockIdx.y.
__global__ __launch_bounds__(kTileBlock) void k_tiles_split_stats(TileArgs a, TileSplit sp) {
    __shared__ int wst[5 * kMaxCrit * kTileWaves];
    const int s = blockIdx.x;
    const long long t = blockIdx.y;
    const int N = a.N, C = a.C, u0 = s * kSplitSlice, u1 = min(N, u0 + kSplitSlice);
    const int *x = a.x + static_cast<size_t>(t) * C * N;
    unsigned long long s2[kMaxCrit];
    int mx[kMaxCrit], mn[kMaxCrit];
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) { s2[c] = 0; mx[c] = -kBig - 1; mn[c] = kBig; }
    for (int u = u0 + threadIdx.x; u < u1; u += kTileBlock) {
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) {
            if (c >= C) break;
            const int e = x[static_cast<size_t>(c) * N + u];
            s2[c] += static_cast<unsigned long long>(static_cast<long long>(e) * e);
            mx[c] = max(mx[c], e);
            mn[c] = min(mn[c], e);
        }
    }
    tile_stats(C, s2, mx, mn, wst);
    if (threadIdx.x < C) {
        const int c = threadIdx.x;
        const size_t o = (static_cast<size_t>(t) * sp.S + s) * C + c;
#pragma unroll
        for (int cc = 0; cc < kMaxCrit; ++cc)
            if (cc == c) { sp.s2[o] = s2[cc]; sp.mx[o] = mx[cc]; sp.mn[o] = mn[cc]; }
    }
}

// grid (S, T): closeness of the slice's servers from the tile's totals, and
// the slice's best feasible key.
__global__ __launch_bounds__(kTileBlock) void k_tiles_split_score(TileArgs a, TileSplit sp) {
    __shared__ unsigned long long ts2[kMaxCrit];
    __shared__ int tmx[kMaxCrit], tmn[kMaxCrit];
    const int s = blockIdx.x;
    const long long t = blockIdx.y;
    const int N = a.N, C = a.C, u0 = s * kSplitSlice, u1 = min(N, u0 + kSplitSlice);
    if (threadIdx.x < C) {
        // tile totals over the slices in slice order (exact integers)
        const int c = threadIdx.x;
        unsigned long long v = 0;
        int hi = -kBig - 1, lo = kBig;
        for (int x = 0; x < sp.S; ++x) {
            const size_t o = (static_cast<size_t>(t) * sp.S + x) * C + c;
            v += sp.s2[o];
            hi = max(hi, sp.mx[o]);
            lo = min(lo, sp.mn[o]);
        }
        ts2[c] = v;
        tmx[c] = hi;
        tmn[c] = lo;
    }
    __syncthreads();
    unsigned long long s2[kMaxCrit];
    int mx[kMaxCrit], mn[kMaxCrit];
#pragma unroll
    for (int c = 0; c < kMaxCrit; ++c) {
        s2[c] = c < C ? ts2[c] : 0;
        mx[c] = c < C ? tmx[c] : 0;
        mn[c] = c < C ? tmn[c] : 0;
    }
    float q[kMaxCrit], ap[kMaxCrit], am[kMaxCrit];
    tile_factors(a, s2, mx, mn, q, ap, am);
    const int *x = a.x + static_cast<size_t>(t) * C * N;
    unsigned long long kb = 0;
    for (int u = u0 + threadIdx.x; u < u1; u += kTileBlock) {
        int vv[kMaxCrit];
#pragma unroll
        for (int c = 0; c < kMaxCrit; ++c) vv[c] = c < C ? x[static_cast<size_t>(c) * N + u] : 0;
        const float sc = topsis_close(C, [&](int c) { return vv[c]; }, q, ap, am);
        if (!a.feas || a.feas[static_cast<size_t>(t) * N + u]) {
            const unsigned long long k = score_key(sc, u);
            kb = k > kb ? k : kb;
        }
        if (a.scores) a.scores[static_cast<size_t>(t) * N + u] = sc;
    }
    kb = tile_block_max<kTileWaves>(kb);
    if (threadIdx.x == 0) sp.key[static_cast<size_t>(t) * sp.S + s] = kb;
}

// grid T, one wave: the tile's best key over its slices.
__global__ __launch_bounds__(kWave) void k_tiles_split_select(TileArgs a, TileSplit sp) {
    const long long t = blockIdx.x;
    unsigned long long kb = 0;
    for (int x = threadIdx.x; x < sp.S; x += kWave) {
        const unsigned long long k = sp.key[static_cast<size_t>(t) * sp.S + x];
        kb = k > kb ? k : kb;
    }
    kb = tile_block_max<1>(kb);
    if (threadIdx.x == 0) tile_write_best(a, t, kb);
}

}  // namespace dcs
