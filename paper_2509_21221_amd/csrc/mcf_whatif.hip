// What-if node addition (paper Sec. VI, handling joining nodes): build the
// batch of instances that tries every assignment of the candidate nodes to
// stages, and reduce solved batches to the best assignment.
//
// Expansion is a pure copy with per-element selection.  A workgroup writes
// up to kExpandPer consecutive placements: one thread each decodes a placement's
// index into its stage -> candidate table in LDS (64-bit divisions, a chain of
// about 0.7 us that one placement per workgroup could not hide), then every
// element's position and base value are worked out once and stored for all of
// them, consecutive lanes on consecutive elements.  The base instance and the
// candidate arrays are small and served from L2; the HBM traffic is the
// instances written.  40,320 placements of 8 x 13 (229 MB): 175 us one
// per workgroup, 88 us (2.6 TB/s) with eight; 11,880 of 12 x 9: 51 and 31 us.
// What bounds it now is issue: one 4-byte store and its address per element.
#include "mcf_internal.h"

#include <algorithm>

namespace gwtf {

namespace {

constexpr int kExpandThreads = 256;
constexpr int kExpandPer = 8;          // placements per workgroup, at most
constexpr int kExpandPerStages = 64;   // longer pipelines: one (the tables would take too much LDS)
constexpr int kExpandBlocks = 1024;    // fewer placements per workgroup rather than fewer workgroups
constexpr int kBestThreads = 1024;

__global__ void __launch_bounds__(kExpandThreads) whatif_expand_kernel(WhatifExpandParams p, int32_t count, int32_t per)
{
    extern __shared__ __align__(8) unsigned char lds[];
    const int S = p.S, n = p.n, m = p.m, slot = p.slot, words = (S + 63) / 64;
    uint64_t *all_used = reinterpret_cast<uint64_t *>(lds);                       // [per][words]
    int32_t *all_at = reinterpret_cast<int32_t *>(lds + 8 * size_t(per) * words); // [per][S]
    const int r0 = int(blockIdx.x) * per, here = min(per, count - r0);

    for (int k = threadIdx.x; k < per * S; k += blockDim.x) all_at[k] = -1;
    for (int w = threadIdx.x; w < per * words; w += blockDim.x) all_used[w] = 0;
    __syncthreads();
    if (int(threadIdx.x) < here) {
        uint64_t *used = all_used + threadIdx.x * words;
        int32_t *at_stage = all_at + threadIdx.x * S;
        // Mixed-radix digits of the placement's index: candidate c picks among
        // the S - c stages still free, and each choice is followed by
        // P(S-c-1, m-c-1) completions (the radix, built from the last
        // candidate back).
        int64_t radix = 1;
        for (int c = m - 1; c > 0; --c) radix *= int64_t(S - c);
        int64_t rem = p.first + r0 + threadIdx.x;
        for (int c = 0; c < m; ++c) {
            int64_t d = rem / radix;
            rem -= d * radix;
            if (c + 1 < m) radix /= int64_t(S - c - 1);
            // stage = the d-th free stage (0-based) in increasing order; the
            // host guarantees r < S!/(S-m)!, so d < S - c free stages remain
            // and the search ends inside the last word at the latest.
            int w = 0;
            for (; w < words - 1; ++w) {
                const int64_t free_here = __popcll(~used[w]);
                if (d < free_here) break;
                d -= free_here;
            }
            uint64_t freebits = ~used[w];
            for (int64_t skip = 0; skip < d; ++skip) freebits &= freebits - 1;
            const int bit = __ffsll((unsigned long long)freebits) - 1;
            used[w] |= uint64_t(1) << bit;
            at_stage[64 * w + bit] = c;
        }
    }
    __syncthreads();

    // Sizes of one instance; the host keeps (S-1) n^2 below 2^31, so 32-bit
    // index arithmetic is exact.
    const uint32_t un = uint32_t(n), SN = uint32_t(S) * un, nn = un * un, na = uint32_t(S - 1) * nn;
    int32_t *cap = p.out_cap + size_t(r0) * SN, *ncost = p.out_cost + size_t(r0) * SN;
    for (uint32_t e = threadIdx.x; e < SN; e += blockDim.x) {
        const int k = int(e / un), i = int(e - uint32_t(k) * un);
        const int32_t base_cap = p.cap[e], base_cost = p.cost[e];
        for (int r = 0; r < here; ++r) {
            const int c = i == slot ? all_at[r * S + k] : -1;
            cap[size_t(r) * SN + e] = c >= 0 ? p.ccap[size_t(c) * S + k] : base_cap;
            ncost[size_t(r) * SN + e] = c >= 0 ? p.ccost[size_t(c) * S + k] : base_cost;
        }
    }
    if (S > 1) {
        int32_t *arc = p.out_arc + size_t(r0) * na;
        for (uint32_t e = threadIdx.x; e < na; e += blockDim.x) {
            const int k = int(e / nn);
            const uint32_t q = e - uint32_t(k) * nn;
            const int i = int(q / un), j = int(q - uint32_t(i) * un);
            const int32_t base = p.arc[e];
            if (i != slot && j != slot) {
                for (int r = 0; r < here; ++r) arc[size_t(r) * na + e] = base;
                continue;
            }
            for (int r = 0; r < here; ++r) {
                const int32_t *at_stage = all_at + r * S;
                const int ci = (i == slot) ? at_stage[k] : -1;     // candidate sending
                const int cj = (j == slot) ? at_stage[k + 1] : -1; // candidate receiving
                int32_t v = base;
                if (ci >= 0 && cj >= 0) v = p.clink[size_t(ci) * m + cj];
                else if (ci >= 0) v = p.cout[(size_t(ci) * S + k) * n + j];
                else if (cj >= 0) v = p.cin[(size_t(cj) * S + k + 1) * n + i];
                arc[size_t(r) * na + e] = v;
            }
        }
    }
    for (int e = threadIdx.x; e < here * n; e += blockDim.x) {
        const int r = e / n, i = e - r * n;
        const int32_t *at_stage = all_at + r * S;
        const int c0 = (i == slot) ? at_stage[0] : -1, cl = (i == slot) ? at_stage[S - 1] : -1;
        p.out_src[size_t(r0) * n + e] = c0 >= 0 ? (p.csrc ? p.csrc[c0] : 0) : (p.src ? p.src[i] : 0);
        p.out_snk[size_t(r0) * n + e] = cl >= 0 ? (p.csnk ? p.csnk[cl] : 0) : (p.snk ? p.snk[i] : 0);
    }
    if (int(threadIdx.x) < here) p.out_supply[size_t(r0) + threadIdx.x] = p.supply[0];
}

// Candidate key: valid, larger F, smaller cost, smaller index wins.
struct Key {
    int64_t idx, F, cost; // idx < 0: no candidate
};

__device__ inline bool better(const Key &a, const Key &b)
{
    if (a.idx < 0) return false;
    if (b.idx < 0) return true;
    if (a.F != b.F) return a.F > b.F;
    if (a.cost != b.cost) return a.cost < b.cost;
    return a.idx < b.idx;
}

__global__ void __launch_bounds__(kBestThreads) whatif_best_kernel(int32_t count, const int64_t *F,
                                                                   const int64_t *cost, const int32_t *status,
                                                                   int64_t first, int32_t merge, int64_t *best)
{
    __shared__ Key part[kBestThreads / 64];
    Key k{-1, 0, 0};
    // eight placements per thread and round, their reads in flight together
    // (one after another, 40,320 placements took 39 us; 29 us now)
    constexpr int kReads = 8;
    for (int64_t at = threadIdx.x; at < count; at += int64_t(kReads) * kBestThreads) {
        Key c[kReads];
        int32_t bad[kReads];
#pragma unroll
        for (int u = 0; u < kReads; ++u) {
            const int64_t i = at + int64_t(u) * kBestThreads, q = i < count ? i : at;
            bad[u] = i < count ? status[q] : 1;
            c[u] = Key{first + q, F[q], cost[q]};
        }
#pragma unroll
        for (int u = 0; u < kReads; ++u)
            if (bad[u] == 0 && better(c[u], k)) k = c[u];
    }
    for (int off = 32; off > 0; off >>= 1) {
        Key o;
        o.idx = __shfl_xor(k.idx, off);
        o.F = __shfl_xor(k.F, off);
        o.cost = __shfl_xor(k.cost, off);
        if (better(o, k)) k = o;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) part[wave] = k;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < int(blockDim.x >> 6); ++w)
            if (better(part[w], k)) k = part[w];
        if (merge) {
            const Key prev{best[0], best[1], best[2]};
            if (better(prev, k)) k = prev;
        }
        if (k.idx < 0) k = Key{-1, 0, 0};
        best[0] = k.idx;
        best[1] = k.F;
        best[2] = k.cost;
    }
}

} // namespace

hipError_t launch_whatif_expand(const WhatifExpandParams &p, int32_t count, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    const int per = p.S <= kExpandPerStages ? std::min(kExpandPer, std::max(1, count / kExpandBlocks)) : 1;
    const size_t lds = size_t(per) * (8 * size_t((p.S + 63) / 64) + 4 * size_t(p.S));
    const int64_t blocks = (int64_t(count) + per - 1) / per;
    hipLaunchKernelGGL(whatif_expand_kernel, dim3(unsigned(blocks)), dim3(kExpandThreads), lds, s, p, count, per);
    return hipGetLastError();
}

hipError_t launch_whatif_best(int32_t count, const int64_t *F, const int64_t *cost, const int32_t *status,
                              int64_t first, int32_t merge, int64_t *best, hipStream_t s)
{
    hipLaunchKernelGGL(whatif_best_kernel, dim3(1), dim3(kBestThreads), 0, s, count, F, cost, status, first,
                       merge, best);
    return hipGetLastError();
}

} // namespace gwtf
