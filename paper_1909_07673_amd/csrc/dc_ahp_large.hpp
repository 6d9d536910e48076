// AHP on the 1-9 scale beyond 8,192 servers (section V-B, Eqs. (9)-(10)):
// the row sums are taken in FP32 over all servers in index order, in the
// chunks and interleaved partial sums of k_ahp_rowsum, so scores are the
// same bit for bit; what is saved is how the terms come about.
//   * Servers of equal value have equal rows: a row is summed once per
//     distinct value (a few dozen for CPU and hops, some 17,000 for 27,648
//     uplinks) instead of once per server.
//   * Column sums are exact integers, so counts replace the pairwise pass.
//   * A wave takes distinct values next to one another in value.  Against
//     one column their entries take one or two neighbouring levels of the
//     scale, so an entry is one compare and one select instead of the 18
//     instructions of the mapping.
// At 27,648 servers and five criteria the pairwise passes took 3.4 ms per
// step that scored, bound by VALU issue; a queue of three requests went from
// 181 to 10.9 ms.  What bounds it now is still VALU issue in k_ahp_rows: three
// instructions per distinct value and column, and some ninety per column.
#pragma once
#include "dc_queue.hpp"

namespace dcs {

// Distinct values per wave.  Thirty-two neighbours of some thousands span a
// level or two of the scale against nearly every column, and a column's
// levels are found once for all of them (a queue at 27,648 servers took 12.4
// ms at 16, 10.8 at 32, 10.6 at 48, 11.3 at 64, where the blocks that span
// more levels keep a few waves busy to the end).  The values of a criterion
// with few are far apart, and only the number of waves counts: with 32 a wave
// too, the same queue took 15.1 ms.
constexpr int kRowBlock = 32, kRowBlockFew = 4, kRowFew = 1024;
constexpr int kRowWaves = 4;         // waves per workgroup, each with its own chunks
constexpr int kRowChunks = 8;        // column chunks per wave: lane = chunk * kAhpAcc + partial sum
static_assert(kRowChunks * kAhpAcc == kWave, "a lane per chunk and partial sum");

struct AhpLarge {
    float *sinv;             // [C][N] 1 / column sum
    int *didx;               // [C][N] index of a server's value among the distinct ones
    int *dist;               // [C][N] distinct values, ascending
    int *count;              // [C] how many
    double *lsum;            // [C][N] row sum of each distinct value
    int vmax[kMaxCrit];      // largest value of each criterion, from the capacities
    int first[kMaxCrit + 1]; // first workgroup of each criterion's row sums
    int groups;              // workgroups per row block (kRowWaves * kRowChunks chunks each)
};

// LDS of the counting kernel: positions (16 bits a value), presence bits and
// their running count.
__host__ __device__ inline size_t large_fwords(int V) { return align4((static_cast<size_t>(V) + 3) >> 1); }
__host__ __device__ inline size_t large_bwords(int V) { return align4((static_cast<size_t>(V) >> 5) + 1); }
inline size_t large_count_lds(int V) { return sizeof(int) * (large_fwords(V) + 2 * large_bwords(V)); }

// Counts of a criterion's values, its column sums and its distinct values.
// Grid (ceil(N / 1024), C): every workgroup counts all servers (the counting
// is short beside another launch) and finishes its own 1,024.  N < 2^16.
__global__ __launch_bounds__(kAhpQueueBlock) void k_ahp_count(Params p, AhpLarge a) {
    extern __shared__ __align__(16) int lds[];
    if (p.b.status[p.s.r] == 0) return;
    constexpr int BS = kAhpQueueBlock, U = 4;
    __shared__ int slots[2][kMaxWaves];
    const int N = p.t.N, c = blockIdx.y, V = a.vmax[c], tid = threadIdx.x, lane = tid & (kWave - 1);
    const int fw = static_cast<int>(large_fwords(V)), bw = static_cast<int>(large_bwords(V));
    unsigned *F = reinterpret_cast<unsigned *>(lds), *bits = F + fw, *before = bits + bw;
    unsigned short *F16 = reinterpret_cast<unsigned short *>(F);
    const int *x = p.xs + static_cast<size_t>(c) * N;
    for (int q = tid; q < fw + 2 * bw; q += BS) F[q] = 0;
    __syncthreads();
    for (int base = 0; base < N; base += U * BS) {
        int v[U];
#pragma unroll
        for (int e = 0; e < U; ++e) v[e] = base + e * BS + tid < N ? x[base + e * BS + tid] : -1;
#pragma unroll
        for (int e = 0; e < U; ++e) {
            // servers with the wave's first value count as one
            const int v0 = uniform(v[e]);
            const bool same = v[e] >= 0 && v[e] == v0;
            const unsigned long long m = __ballot(same);
            const bool first = same && lane == __builtin_ctzll(m);
            const unsigned cnt = first ? static_cast<unsigned>(__builtin_popcountll(m)) : 1u;
            if (v[e] >= 0 && (!same || first)) atomicAdd(F + (v[e] >> 1), cnt << (16 * (v[e] & 1)));
        }
    }
    __syncthreads();
    // presence bits: a wave reads 64 counts and writes two words
    for (int q = 2 * (tid / kWave); q < bw; q += 2 * (BS / kWave)) {
        const int v = 32 * q + lane;
        const unsigned long long m = __ballot(v <= V && F16[min(v, V)] != 0);
        if (lane < 2 && q + lane < bw) bits[q + lane] = static_cast<unsigned>(m >> (32 * lane));
    }
    __syncthreads();
    {
        const int per = (bw + BS - 1) / BS, w0 = min(bw, tid * per), w1 = min(bw, w0 + per);
        int sum = 0, total;
        for (int q = w0; q < w1; ++q) sum += __builtin_popcount(bits[q]);
        int at = block_scan<BS>(sum, slots[0], total);
        for (int q = w0; q < w1; ++q) {
            before[q] = at;
            at += __builtin_popcount(bits[q]);
        }
        if (blockIdx.x == 0 && tid == 0) a.count[c] = total;
    }
    // counts to positions (odd runs: the threads start in different banks)
    {
        const int per = ((fw + BS - 1) / BS) | 1, w0 = min(fw, tid * per), w1 = min(fw, w0 + per);
        int sum = 0, total;
        for (int q = w0; q < w1; ++q) sum += static_cast<int>((F[q] & 0xffffu) + (F[q] >> 16));
        unsigned at = block_scan<BS>(sum, slots[1], total);
        for (int q = w0; q < w1; ++q) {
            const unsigned o = F[q], hi = at + (o & 0xffffu);
            F[q] = at | hi << 16;
            at = hi + (o >> 16);
        }
    }
    __syncthreads();
    const int u = blockIdx.x * BS + tid;
    if (u >= N) return;
    const int v = x[u];
    const SaatyBuckets b = saaty_positions(v, V, N, [&](int t) { return static_cast<int>(F16[t]); });
    const int cs = saaty_sum<int>(b, N, p.m.cost[c] != 0, [](int lo, int hi) { return hi - lo; });
    const size_t at = static_cast<size_t>(c) * N;
    const int idx = static_cast<int>(before[v >> 5]) + __builtin_popcount(bits[v >> 5] & ((1u << (v & 31)) - 1));
    a.sinv[at + u] = static_cast<float>(1.0 / static_cast<double>(cs));
    a.didx[at + u] = idx;
    a.dist[at + idx] = v;                       // servers of equal value write the same
}

// Level of p against q on the scale, ascending in p: s - 1 when p >= q, 1 - s
// below (s the rounded ratio as in saaty2520).
__device__ __forceinline__ float saaty_level(float p, float q, float rp, float rq) {
    const bool ge = p >= q;
    const float hi = ge ? p : q, lo = ge ? q : p, rl = ge ? rq : rp;
    const float num = fmaf(2.f, hi, lo), two_lo = lo + lo;
    float s = floorf(num * rl);
    const float rem = fmaf(-s, two_lo, num);
    s = fminf(rem >= two_lo ? s + 1.f : s, 9.f);
    return ge ? s - 1.f : 1.f - s;
}

// 2520 times the entry at a level.
__device__ __forceinline__ float level2520(float l) {
    const float s = fabsf(l) + 1.f;
    return rintf(2520.f * (l >= 0.f ? s : __builtin_amdgcn_rcpf(s)));
}

// Smallest integer p whose level against q is at least l (-7 <= l <= 8, q > 0
// where l > 0): the ratio p / q rounds to l + 1 from (2l + 1) q / 2 on, and
// q / p rounds to at most 1 - l beyond 2q / (3 - 2l).
__device__ __forceinline__ float level_from(float l, float q) {
    if (l > 0.f) return floorf(fmaf(2.f * l + 1.f, q, 1.f) * 0.5f);   // integers below 2^24 + ..: exact to l = 1..8
    const float d = 3.f - 2.f * l, n = 2.f * q;
    float f = floorf(n * __builtin_amdgcn_rcpf(d));
    float r = fmaf(-f, d, n);
    f = r < 0.f ? f - 1.f : r >= d ? f + 1.f : f;
    return f + 1.f;
}

// Row sums of R distinct values of criterion c over kRowChunks chunks per
// wave.  Lane (chunk, a) carries partial sum a of its chunk for all R rows;
// the rows' values are the same on every lane.  at: the workgroup's number
// within the criterion; part: R rows of LDS per wave.
template <int R>
__device__ __forceinline__ void row_block(const Params &p, const AhpLarge &a, int c, int at, float (*part)[kWave + 1]) {
    const int N = p.t.N, r0 = at / a.groups * R, D = uniform(a.count[c]);
    if (r0 >= D) return;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int ck0 = (at % a.groups * kRowWaves + wid) * kRowChunks;
    if (ck0 >= p.nJ) return;                    // (no workgroup barrier below)
    const size_t row = static_cast<size_t>(c) * N;
    const float sign = p.m.cost[c] ? -1.f : 1.f;    // a cost criterion compares q with p
    int pv[R];                          // in scalar registers
#pragma unroll
    for (int r = 0; r < R; ++r) pv[r] = uniform(a.dist[row + min(r0 + r, D - 1)]);
    const float pmin = static_cast<float>(pv[0]), pmax = static_cast<float>(pv[R - 1]);
    const float rmin = rcp2(pmin), rmax = rcp2(pmax);
    // the columns of this lane's chain: every eighth of the chunk, and for
    // partial sum 0 the chunk's tail after them
    const int ck = ck0 + lane / kAhpAcc, al = lane % kAhpAcc;
    const int j0 = ck * p.tj, cnt = ck < p.nJ ? min(p.tj, N - j0) : 0;
    const int main8 = cnt / kAhpAcc, len = main8 + (al == 0 ? cnt - main8 * kAhpAcc : 0);
    const int steps = wave_max(len);
    const int *x = p.xs + row;
    const float *sv = a.sinv + row;
    auto column = [&](int t) {
        return t >= len ? 0 : t < main8 ? j0 + t * kAhpAcc + al : j0 + main8 * kAhpAcc + (t - main8);
    };
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.f;
    int j = column(0);
    int xn = x[j];
    float sn = sv[j];
    for (int t = 0; t < steps; ++t) {
        const bool in = t < len;
        const float q = static_cast<float>(xn), si = in ? sn : 0.f;      // si = 0 adds nothing
        j = column(t + 1);
        xn = x[j];
        sn = sv[j];
        const float rq = rcp2(q);
        const float llo = saaty_level(pmin, q, rmin, rq);
        const float lhi = in ? saaty_level(pmax, q, rmax, rq) : llo;
        if (__all(lhi == llo)) {
            const float e = level2520(sign * llo);
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fmaf(e, si, acc[r]);
        } else if (__all(lhi - llo <= 1.f)) {
            const float elo = level2520(sign * llo), ehi = level2520(sign * lhi);
            const int from = static_cast<int>(level_from(lhi, q));
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fmaf(pv[r] >= from ? ehi : elo, si, acc[r]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                int o = pv[r];
                asm volatile("" : "+s"(o));            // the reciprocals are not worth 64 registers
                const float pr = static_cast<float>(o), rp = rcp2(pr);
                acc[r] = fmaf(level2520(sign * saaty_level(pr, q, rp, rq)), si, acc[r]);
            }
        }
    }
    // a chunk's sum: its partial sums in order, through LDS (each wave its own)
#pragma unroll
    for (int r = 0; r < R; ++r) part[r][lane] = acc[r];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int it = lane; it < R * kRowChunks; it += kWave) {
        const int r = it % R, k = it / R;
        float s = 0.f;
#pragma unroll
        for (int b = 0; b < kAhpAcc; ++b) s += part[r][k * kAhpAcc + b];
        if (r0 + r < D && ck0 + k < p.nJ) p.rowpart[(static_cast<size_t>(c) * p.nJ + ck0 + k) * N + r0 + r] = s;
    }
}

// Workgroups first[c] .. first[c + 1] - 1 take criterion c's row blocks, of
// as many values as it can have; those past the values it has leave.
__global__ __launch_bounds__(kRowWaves *kWave) void k_ahp_rows(Params p, AhpLarge a) {
    if (p.b.status[p.s.r] == 0) return;
    __shared__ float part[kRowWaves][kRowBlock][kWave + 1];
    int c = 0;
    while (c + 1 < p.m.nc && static_cast<int>(blockIdx.x) >= a.first[c + 1]) ++c;
    const int at = blockIdx.x - a.first[c], wid = threadIdx.x / kWave;
    if (a.vmax[c] < kRowFew) row_block<kRowBlockFew>(p, a, c, at, part[wid]);
    else row_block<kRowBlock>(p, a, c, at, part[wid]);
}

// Row sum of each distinct value over the chunks, in order.
__global__ __launch_bounds__(kAhpBlock) void k_ahp_row_total(Params p, AhpLarge a) {
    if (p.b.status[p.s.r] == 0) return;
    const int N = p.t.N, c = blockIdx.y, i = blockIdx.x * kAhpBlock + threadIdx.x;
    if (i >= a.count[c]) return;
    double l = 0.0;
#pragma unroll 8
    for (int jb = 0; jb < p.nJ; ++jb) l += p.rowpart[(static_cast<size_t>(c) * p.nJ + jb) * N + i];
    a.lsum[static_cast<size_t>(c) * N + i] = l;
}

}  // namespace dcs
