// Batched simulation of GWTF's decentralized flow heuristic (paper Sec. V-C:
// Request Flow, Request Change, Request Redirect under simulated annealing;
// Sec. VI setup: T0 = 1.7, alpha = 0.95), for scoring it against the exact
// optimum the solver passes compute (Sec. VI flow ablation).
//
// One wave per instance, one lane per relay node (S * n <= 64).  The instance
// lives in LDS: link costs, node arrays, and one slot per unit of capacity
// (a slot holds one microbatch: its outflow to the next hop's slot or to the
// data node D, and its inflow from the previous hop's slot or from D).
// Rounds are synchronous:
//   1. cost to the sink of every used slot, from the last stage to the first;
//   2. Request Flow: every relay with no unpaired outflow and a free slot
//      asks the next-stage relay whose unpaired outflow minimises its cost to
//      the sink plus the link cost (lowest index on ties); a target approves
//      its lowest-index requester, D as sink its requesters in index order
//      while it has flow left; D as source pairs first-stage unpaired
//      outflows cheapest first (source link plus cost to the sink);
//   3. improvement: stages of even index, then odd ones, each shuffled and
//      split into pairs (proposer, partner); a proposer that sent no Request
//      Flow this round draws a Request Redirect (carry one of the partner's
//      paired flows itself) or a Request Change (swap next hops of one flow
//      each) and takes it when exp((cost_cur - cost_new) / T) > U(0, 1),
//      with Eq. 1 link costs summed or maximised; an accepted move cools the
//      proposer's T by alpha.
// Moves of different pairs touch disjoint slots, and a stage's moves touch
// only the in-links of the next stage's slots and the out-links of the
// previous stage's, so all pairs of all stages of one parity run at once.
// Random numbers: Philox4x64-10 (Salmon et al., SC 2011) with key (seed,
// instance) and counter (round, stage, stream, index): stream 0 drives the
// stage's Fisher-Yates shuffle, stream 1 pair m's four draws.  The result is
// the set of complete paths (slot chains from D back to D): their number F,
// their Eq. 2 cost, and their node and link flows.
//
// heuristic_kernel keeps each relay's slots as masks of 32 bits; instances
// with a relay of more slots go on to heuristic_general_kernel, which passes
// over the slots and draws its random numbers where it uses them.
#include "mcf_internal.h"

#include <math.h>

#include <utility>

namespace gwtf {
namespace {

constexpr int32_t kSlotNone = -1; // free slot / no inflow yet
constexpr int32_t kData = -2;     // the data node, as source (inflow) or sink (outflow)
constexpr int32_t kNoLink = -1;

// status between the two launches: a relay has more than kMaskSlots slots
constexpr int32_t kPassedOn = -1;
constexpr int kMaskSlots = 32;
constexpr int kChunkRounds = 8; // rounds whose random numbers are drawn together

struct HeurLayout {
    size_t lk, src, snk, cost, cap, base, unp, req, key, perm, owner, sin, sout, cs, total;
};

__host__ __device__ inline HeurLayout heur_layout(int S, int n, int slots)
{
    HeurLayout L;
    const size_t V = size_t(S) * n, nl = size_t(S - 1) * n * n;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align16(o + bytes); return at; };
    L.lk = take(4 * (nl > 0 ? nl : 1));
    L.src = take(4 * size_t(n));
    L.snk = take(4 * size_t(n));
    L.cost = take(4 * V);
    L.cap = take(4 * V);
    L.base = take(4 * (V + 1));
    L.unp = take(4 * V);
    L.req = take(4 * V);
    L.key = take(4 * V);
    L.perm = take(4 * V);
    L.owner = take(size_t(slots));
    L.sin = take(2 * size_t(slots));
    L.sout = take(2 * size_t(slots));
    L.cs = take(4 * size_t(slots));
    L.total = o;
    return L;
}

// Philox4x64-10: ten rounds of two 64 x 64 -> 128-bit products of counter
// words 0 and 2 with fixed multipliers, the key bumped by two Weyl constants
// between rounds.
__device__ inline void philox(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0, uint64_t k1,
                              uint64_t out[4])
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll 1 // rolled: the unrolled rounds cost a wave per SIMD in registers
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += W0;
            k1 += W1;
        }
        const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// A draw in [0, m) from the high 32 bits of a word.
__device__ inline int32_t draw_below(uint64_t w, uint32_t m) { return int32_t(((w >> 32) * uint64_t(m)) >> 32); }

struct Inst {
    int S, n, V;
    int32_t *lk, *src, *snk, *cost, *cap, *base, *unp, *req, *key, *perm, *cs;
    uint8_t *owner;
    int16_t *sin, *sout;

    __device__ int stage(int v) const { return v / n; }
    __device__ int idx(int v) const { return v - (v / n) * n; }
    __device__ int node_at(int32_t slot) const { return slot == kData ? kData : int(owner[slot]); }
    // link cost x -> y (either end may be the data node)
    __device__ int32_t edge(int x, int y) const
    {
        if (x == kData) return src[idx(y)];
        if (y == kData) return snk[idx(x)];
        return lk[(stage(x) * n + idx(x)) * n + idx(y)];
    }
    __device__ int32_t ccost(int x) const { return x == kData ? 0 : cost[x]; }
    // Eq. 1 cost of the link x -> y, doubled: 2 * link + c_x + c_y
    __device__ int64_t E(int x, int y) const { return 2 * int64_t(edge(x, y)) + ccost(x) + ccost(y); }
    __device__ int lowest_free(int v) const
    {
        for (int s = base[v]; s < base[v + 1]; ++s)
            if (sout[s] == kSlotNone) return s;
        return kSlotNone;
    }
    // q-th (from 0) used slot of v, or q-th paired slot when paired_only
    __device__ int nth(int v, int q, bool paired_only) const
    {
        for (int s = base[v]; s < base[v + 1]; ++s) {
            if (sout[s] == kSlotNone || (paired_only && sin[s] == kSlotNone)) continue;
            if (q-- == 0) return s;
        }
        return kSlotNone;
    }
};

__device__ inline int wave_popc(uint64_t m) { return __popcll(m); }

__device__ inline int64_t wave_sum64(int64_t x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ inline int32_t wave_max32(int32_t x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = max(x, __shfl_xor(x, o, 64));
    return x;
}

// Relays of more than 32 slots: what heuristic_kernel passed on.
__global__ void __launch_bounds__(64) heuristic_general_kernel(HeurParams p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int b = blockIdx.x, lane = threadIdx.x;
    if (p.status_out[b] != kPassedOn) return;
    const int S = p.S, n = p.n, V = S * n;
    const int64_t nl = int64_t(S - 1) * n * n;
    const HeurLayout L = heur_layout(S, n, p.max_slots);
    Inst I;
    I.S = S;
    I.n = n;
    I.V = V;
    I.lk = reinterpret_cast<int32_t *>(lds + L.lk);
    I.src = reinterpret_cast<int32_t *>(lds + L.src);
    I.snk = reinterpret_cast<int32_t *>(lds + L.snk);
    I.cost = reinterpret_cast<int32_t *>(lds + L.cost);
    I.cap = reinterpret_cast<int32_t *>(lds + L.cap);
    I.base = reinterpret_cast<int32_t *>(lds + L.base);
    I.unp = reinterpret_cast<int32_t *>(lds + L.unp);
    I.req = reinterpret_cast<int32_t *>(lds + L.req);
    I.key = reinterpret_cast<int32_t *>(lds + L.key);
    I.perm = reinterpret_cast<int32_t *>(lds + L.perm);
    I.owner = lds + L.owner;
    I.sin = reinterpret_cast<int16_t *>(lds + L.sin);
    I.sout = reinterpret_cast<int16_t *>(lds + L.sout);
    I.cs = reinterpret_cast<int32_t *>(lds + L.cs);

    const bool node = lane < V;
    const int v = lane, k = node ? lane / n : 0, i = node ? lane - k * n : 0;

    // ---- ingest and checks ----
    int32_t cap = node ? p.cap[int64_t(b) * V + v] : 0;
    int32_t cst = node ? p.cost[int64_t(b) * V + v] : 0;
    bool bad = node && (cap < 0 || cst < 0);
    int32_t maxc = cst;
    for (int64_t q = lane; q < nl; q += 64) {
        const int32_t w = p.arc[int64_t(b) * nl + q];
        I.lk[q] = w;
        bad |= w < kNoLink;
        maxc = max(maxc, w);
    }
    for (int q = lane; q < n; q += 64) {
        const int32_t a = p.src ? p.src[int64_t(b) * n + q] : 0, z = p.snk ? p.snk[int64_t(b) * n + q] : 0;
        I.src[q] = a;
        I.snk[q] = z;
        bad |= a < 0 || z < 0;
        maxc = max(maxc, max(a, z));
    }
    const int32_t supply = p.supply[b];
    // slot ranges: inclusive scan of the capacities over the lanes
    int64_t incl = node ? max(cap, 0) : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    const int64_t total_cap = __shfl(incl, 63, 64);
    maxc = wave_max32(maxc);
    int32_t status = 0;
    if (__any(bad) || supply < 0 || total_cap > p.max_slots) status = 1;
    else if (int64_t(2 * S + 2) * maxc >= (int64_t(1) << 30)) status = 2;
    int src_left = supply, sink_left = supply;
    if (status == 0) {
        if (node) {
            I.cost[v] = cst;
            I.cap[v] = cap;
            I.base[v] = int32_t(incl - cap);
            for (int s = int(incl - cap); s < int(incl); ++s) {
                I.owner[s] = uint8_t(v);
                I.sin[s] = kSlotNone;
                I.sout[s] = kSlotNone;
            }
        }
        if (lane == 0) I.base[V] = int32_t(total_cap);
        __syncthreads();
        // initial complete paths, laid out in order by lane 0
        if (p.paths && p.num_paths > 0) {
            int32_t ok = 1;
            if (lane == 0) {
                for (int q = 0; q < p.num_paths && ok; ++q) {
                    const int32_t *path = p.paths + (int64_t(b) * p.num_paths + q) * S;
                    if (path[0] < 0) continue;
                    if (src_left <= 0 || sink_left <= 0) {
                        ok = 0;
                        break;
                    }
                    int32_t prev = kData;
                    for (int kk = 0; kk < S && ok; ++kk) {
                        const int32_t j = path[kk];
                        if (j < 0 || j >= n) {
                            ok = 0;
                            break;
                        }
                        const int w = kk * n + j;
                        if (prev != kData && I.edge(I.owner[prev], w) == kNoLink) {
                            ok = 0;
                            break;
                        }
                        const int z = I.lowest_free(w);
                        if (z == kSlotNone) {
                            ok = 0;
                            break;
                        }
                        I.sin[z] = int16_t(prev);
                        I.sout[z] = kData;
                        if (prev != kData) I.sout[prev] = int16_t(z);
                        prev = z;
                    }
                    if (ok) {
                        --src_left;
                        --sink_left;
                    }
                }
            }
            ok = __shfl(ok, 0, 64);
            src_left = __shfl(src_left, 0, 64);
            sink_left = __shfl(sink_left, 0, 64);
            if (!ok) status = 1;
            __syncthreads();
        }
    }

    double T = p.t0;
    int32_t acc = 0;
    int64_t approvals = 0;
    if (status == 0) {
        const uint64_t key0 = p.seed, key1 = uint64_t(b);
        for (int r = 0; r < p.rounds; ++r) {
            // ---- cost to the sink, last stage first; unpaired outflow and
            // used slots of each relay ----
            int32_t unp = kSlotNone, used = 0;
            for (int kk = S - 1; kk >= 0; --kk) {
                if (node && k == kk) {
                    for (int s = I.base[v]; s < I.base[v + 1]; ++s) {
                        const int32_t o = I.sout[s];
                        if (o == kSlotNone) continue;
                        ++used;
                        if (unp == kSlotNone && I.sin[s] == kSlotNone) unp = s;
                        I.cs[s] = cst + I.edge(v, I.node_at(o)) + (o == kData ? 0 : I.cs[o]);
                    }
                    I.unp[v] = unp;
                }
                __syncthreads();
            }
            // ---- Request Flow: choose targets ----
            int32_t req = kSlotNone;
            if (node && unp == kSlotNone && used < cap) {
                if (k == S - 1) {
                    if (sink_left > 0) req = kData;
                } else {
                    int32_t best = 0;
                    for (int j = 0; j < n; ++j) {
                        const int w = (k + 1) * n + j, u = I.unp[w];
                        const int32_t l = I.lk[(k * n + i) * n + j];
                        if (u == kSlotNone || l == kNoLink) continue;
                        const int32_t score = I.cs[u] + l;
                        if (req == kSlotNone || score < best) {
                            best = score;
                            req = w;
                        }
                    }
                }
            }
            if (node) {
                I.req[v] = req;
                I.key[v] = (k == 0 && unp != kSlotNone) ? I.src[i] + I.cs[unp] : 0;
            }
            __syncthreads();
            // approvals: lowest requester per relay target; D as sink in
            // index order while it has flow left
            const uint64_t sink_reqs = __ballot(node && req == kData);
            bool win = false;
            if (req >= 0) {
                win = true;
                for (int q = k * n; q < v; ++q)
                    if (I.req[q] == req) win = false;
            } else if (req == kData) {
                win = wave_popc(sink_reqs & ((uint64_t(1) << v) - 1)) < sink_left;
            }
            // D as source: first-stage unpaired outflows, cheapest first
            bool paired_by_data = false;
            if (node && k == 0 && unp != kSlotNone && src_left > 0) {
                const int32_t mine = I.key[v];
                int rank = 0;
                for (int j = 0; j < n; ++j) {
                    if (j == i || I.unp[j] == kSlotNone) continue;
                    const int32_t other = I.key[j];
                    rank += other < mine || (other == mine && j < i);
                }
                paired_by_data = rank < src_left;
            }
            const int data_pairs = wave_popc(__ballot(paired_by_data));
            const int sink_wins = wave_popc(__ballot(win && req == kData));
            approvals += wave_popc(__ballot(win));
            __syncthreads();
            if (paired_by_data) I.sin[unp] = kData;
            if (win) {
                const int z = I.lowest_free(v);
                if (req == kData) {
                    I.sout[z] = kData;
                } else {
                    const int u = I.unp[req];
                    I.sout[z] = int16_t(u);
                    I.sin[u] = int16_t(z);
                }
                I.sin[z] = kSlotNone;
            }
            src_left -= data_pairs;
            sink_left -= sink_wins;
            __syncthreads();

            // ---- improvement: even stages, then odd ones ----
            const bool improver = node && req == kSlotNone;
            for (int parity = 0; parity < 2; ++parity) {
                const bool active = node && (k & 1) == parity;
                if (active && i == 0) {
                    // Fisher-Yates shuffle of the stage (stream 0)
                    int32_t *pm = I.perm + k * n;
                    for (int j = 0; j < n; ++j) pm[j] = j;
                    uint64_t words[4];
                    int word = 4, block = 0;
                    for (int j = n - 1; j >= 1; --j) {
                        if (word == 4) {
                            philox(uint64_t(r), uint64_t(k), 0, uint64_t(block++), key0, key1, words);
                            word = 0;
                        }
                        const int t = draw_below(words[word++], uint32_t(j + 1));
                        const int32_t x = pm[j];
                        pm[j] = pm[t];
                        pm[t] = x;
                    }
                }
                __syncthreads();
                if (active && improver) {
                    const int32_t *pm = I.perm + k * n;
                    int pos = 0;
                    while (pos < n - 1 && pm[pos] != i) ++pos; // pm is a permutation of 0..n-1
                    if ((pos & 1) == 0 && pos + 1 < n) {
                        const int a = v, bn = k * n + pm[pos + 1], m = pos >> 1;
                        uint64_t w[4];
                        philox(uint64_t(r), uint64_t(k), 1, uint64_t(m), key0, key1, w);
                        int used_a = 0, used_b = 0, paired_b = 0;
                        for (int s = I.base[a]; s < I.base[a + 1]; ++s) used_a += I.sout[s] != kSlotNone;
                        for (int s = I.base[bn]; s < I.base[bn + 1]; ++s) {
                            used_b += I.sout[s] != kSlotNone;
                            paired_b += I.sout[s] != kSlotNone && I.sin[s] != kSlotNone;
                        }
                        const bool can_redirect = used_a < cap && paired_b > 0;
                        const bool can_change = used_a > 0 && used_b > 0;
                        if (can_redirect || can_change) {
                            const bool redirect = can_redirect && can_change ? (w[0] & 1) != 0 : can_redirect;
                            const double U = double(w[3] >> 11) * (1.0 / 9007199254740992.0);
                            if (redirect) {
                                const int y = I.nth(bn, draw_below(w[1], uint32_t(paired_b)), true);
                                const int32_t up = I.sin[y], dn = I.sout[y];
                                const int un = I.node_at(up), dw = I.node_at(dn);
                                if (I.edge(un, a) != kNoLink && I.edge(a, dw) != kNoLink) {
                                    const int64_t c0 = I.E(un, bn), c1 = I.E(bn, dw), n0 = I.E(un, a), n1 = I.E(a, dw);
                                    const int64_t cur = p.objective ? max(c0, c1) : c0 + c1;
                                    const int64_t nxt = p.objective ? max(n0, n1) : n0 + n1;
                                    if (exp(double(cur - nxt) * 0.5 / T) > U) {
                                        const int z = I.lowest_free(a);
                                        I.sin[z] = int16_t(up);
                                        I.sout[z] = int16_t(dn);
                                        if (up != kData) I.sout[up] = int16_t(z);
                                        if (dn != kData) I.sin[dn] = int16_t(z);
                                        I.sin[y] = kSlotNone;
                                        I.sout[y] = kSlotNone;
                                        T *= p.alpha;
                                        ++acc;
                                    }
                                }
                            } else {
                                const int x = I.nth(a, draw_below(w[1], uint32_t(used_a)), false);
                                const int y = I.nth(bn, draw_below(w[2], uint32_t(used_b)), false);
                                const int32_t ox = I.sout[x], oy = I.sout[y];
                                const int nx = I.node_at(ox), ny = I.node_at(oy);
                                if (nx != ny && I.edge(a, ny) != kNoLink && I.edge(bn, nx) != kNoLink) {
                                    const int64_t c0 = I.E(a, nx), c1 = I.E(bn, ny), n0 = I.E(a, ny), n1 = I.E(bn, nx);
                                    const int64_t cur = p.objective ? max(c0, c1) : c0 + c1;
                                    const int64_t nxt = p.objective ? max(n0, n1) : n0 + n1;
                                    if (exp(double(cur - nxt) * 0.5 / T) > U) {
                                        I.sout[x] = int16_t(oy);
                                        I.sout[y] = int16_t(ox);
                                        if (oy != kData) I.sin[oy] = int16_t(x);
                                        if (ox != kData) I.sin[ox] = int16_t(y);
                                        T *= p.alpha;
                                        ++acc;
                                    }
                                }
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
    }

    // ---- result: complete paths, stage by stage from the source ----
    int32_t nf = 0, used = 0;
    int64_t mycost = 0;
    if (status == 0) {
        int32_t *complete = I.cs; // cost to the sink is no longer needed
        for (int kk = 0; kk < S; ++kk) {
            if (node && k == kk) {
                for (int s = I.base[v]; s < I.base[v + 1]; ++s) {
                    const int32_t o = I.sout[s], in = I.sin[s];
                    int32_t c = 0;
                    if (o != kSlotNone) {
                        ++used;
                        c = in == kData || (in >= 0 && complete[in]);
                        if (c) {
                            ++nf;
                            mycost += cst + I.edge(v, I.node_at(o)) + (k == 0 ? I.src[i] : 0);
                        }
                    }
                    complete[s] = c;
                }
            }
            __syncthreads();
        }
    }
    const int64_t F = wave_sum64(node && k == 0 ? nf : 0);
    const int64_t cost = wave_sum64(mycost);
    const int64_t accepted = wave_sum64(acc);
    const int64_t dangling = wave_sum64(used - nf);
    if (lane == 0) {
        p.F_out[b] = status == 0 ? F : 0;
        p.cost_out[b] = status == 0 ? cost : 0;
        p.status_out[b] = status;
        if (p.counters) {
            int64_t *c = p.counters + int64_t(b) * 4;
            c[0] = status == 0 ? supply - src_left : 0;
            c[1] = status == 0 ? approvals : 0;
            c[2] = status == 0 ? accepted : 0;
            c[3] = status == 0 ? dangling : 0;
        }
    }
    if (node) {
        const int64_t at = int64_t(b) * V + v;
        if (p.node_flow) p.node_flow[at] = nf;
        if (p.used) p.used[at] = used;
        if (p.accepted) p.accepted[at] = acc;
        if (p.temperature) p.temperature[at] = T;
        if (p.arc_flow && k < S - 1) {
            int32_t *row = p.arc_flow + (int64_t(b) * (S - 1) + k) * n * n + int64_t(i) * n;
            for (int j = 0; j < n; ++j) {
                int32_t cnt = 0;
                if (status == 0)
                    for (int s = I.base[v]; s < I.base[v + 1]; ++s) {
                        const int32_t o = I.sout[s];
                        cnt += o >= 0 && I.cs[s] && I.idx(I.owner[o]) == j;
                    }
                row[j] = cnt;
            }
        }
    }
}

// LDS of heuristic_kernel: link costs, node arrays, per relay the masks of its
// used and of its paired slots, per slot its owner, inflow and {cost of its
// relay and outgoing link, outflow}, and the random numbers of a chunk of
// rounds: per pair {slot draws, U word with the move bit in bit 0}, per relay
// its partner | pair << 8 (kNoPair when it proposes nothing), and room for the
// shuffles.
struct MaskLayout {
    size_t lk, src, snk, cost, base, used, paired, head, win, slot, pairs, partner, sin, perm, owner, total;
};
struct PairDraw {
    uint32_t w1, w2;
    uint64_t w3;
};
constexpr uint32_t kNoPair = 0xffff;
constexpr int32_t kNoHead = 0x7fffffff;

__host__ __device__ inline MaskLayout mask_layout(int S, int n, int max_slots)
{
    MaskLayout L;
    // relays of at most kMaskSlots slots hold no more than this together
    const int slots = max_slots < kMaskSlots * S * n ? max_slots : kMaskSlots * S * n;
    const size_t V = size_t(S) * n, nl = size_t(S - 1) * n * n;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align16(o + bytes); return at; };
    L.slot = take(8 * size_t(slots));
    L.pairs = take(sizeof(PairDraw) * kChunkRounds * S * (n / 2));
    L.lk = take(4 * nl);
    L.src = take(4 * size_t(n));
    L.snk = take(4 * size_t(n));
    L.cost = take(4 * V);
    L.base = take(4 * V);
    L.used = take(4 * V);
    L.paired = take(4 * V);
    L.head = take(4 * V);
    L.win = take(4 * V);
    L.partner = take(2 * kChunkRounds * V);
    L.sin = take(2 * size_t(slots));
    L.perm = take(kChunkRounds * V);
    L.owner = take(size_t(slots));
    L.total = o;
    return L;
}

// Index of the q-th (from 0) set bit of m.
__device__ inline int nth_bit(uint32_t m, int q)
{
    while (q-- > 0) m &= m - 1;
    return __builtin_ctz(m);
}

// exp((cur - nxt) / (2 T)) > U in IEEE double.  exp of a value >= 0 is at
// least 1 > U.  Otherwise a single-precision estimate decides where it is
// more than a thousandth away from U (its relative error is below 1e-4: the
// argument's rounding, 3 * 2^-24 of at most 104 before the estimate is 0, and
// the exponential's own); the double value decides the rest.
__device__ inline bool accepts(int32_t cur, int32_t nxt, double T, double U)
{
    if (cur >= nxt && T > 0.0) return true;
    const float est = __expf(float(cur - nxt) * 0.5f / float(T)), u = float(U);
    if (cur < nxt && u > 1e-20f) {
        if (est > u * 1.001f) return true;
        if (est < u * 0.999f) return false;
    }
    return exp(double(cur - nxt) * 0.5 / T) > U;
}

// The simulation with slot masks, one wave per instance.  What bounds it is
// VALU issue, so what does not depend on the state is taken out of the rounds:
// the random numbers of eight rounds are drawn at once with all lanes busy
// (one Philox block per lane; drawn where they are used, a block kept 4 to 10
// lanes busy and a round took four), and with them the shuffles, which leave
// every relay its partner.  A relay's slots are two 32-bit masks, so counting,
// the lowest free and the q-th used slot take a few instructions instead of a
// pass over the slots; and a slot keeps the cost of its relay and outgoing
// link, so that only the heads of unpaired chains, the one place a cost to
// the sink is read from, walk their chain.  16,384 instances of 8 x 5, 120
// rounds: 11.3 ms before, 1.82 ms now (six waves per SIMD with a few spilled
// registers; 2.10 at four without, 1.93 at five, 2.07 at eight).
__global__ void __launch_bounds__(64, 6) heuristic_kernel(HeurParams p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int b = blockIdx.x, lane = threadIdx.x;
    const int S = p.S, n = p.n, V = S * n, half = n / 2;
    const int nl = (S - 1) * n * n;
    const MaskLayout L = mask_layout(S, n, p.max_slots);
    int32_t *lk = reinterpret_cast<int32_t *>(lds + L.lk), *src = reinterpret_cast<int32_t *>(lds + L.src);
    int32_t *snk = reinterpret_cast<int32_t *>(lds + L.snk), *cost = reinterpret_cast<int32_t *>(lds + L.cost);
    int32_t *base = reinterpret_cast<int32_t *>(lds + L.base), *head = reinterpret_cast<int32_t *>(lds + L.head);
    int32_t *winner = reinterpret_cast<int32_t *>(lds + L.win);
    uint32_t *usedm = reinterpret_cast<uint32_t *>(lds + L.used), *pairedm = reinterpret_cast<uint32_t *>(lds + L.paired);
    int2 *slot = reinterpret_cast<int2 *>(lds + L.slot); // {relay + link cost, outflow}
    int16_t *sin = reinterpret_cast<int16_t *>(lds + L.sin);
    uint8_t *owner = lds + L.owner, *perm = lds + L.perm;
    PairDraw *pairs = reinterpret_cast<PairDraw *>(lds + L.pairs);
    uint16_t *partner = reinterpret_cast<uint16_t *>(lds + L.partner);

    const bool node = lane < V;
    const int v = lane, k = node ? lane / n : 0, i = node ? lane - k * n : 0;

    // ---- ingest and checks ----
    const int32_t cap = node ? p.cap[int64_t(b) * V + v] : 0;
    const int32_t cst = node ? p.cost[int64_t(b) * V + v] : 0;
    bool bad = node && (cap < 0 || cst < 0);
    int32_t maxc = cst;
    for (int q = lane; q < nl; q += 64) {
        const int32_t w = p.arc[int64_t(b) * nl + q];
        lk[q] = w;
        bad |= w < kNoLink;
        maxc = max(maxc, w);
    }
    for (int q = lane; q < n; q += 64) {
        const int32_t a = p.src ? p.src[int64_t(b) * n + q] : 0, z = p.snk ? p.snk[int64_t(b) * n + q] : 0;
        src[q] = a;
        snk[q] = z;
        bad |= a < 0 || z < 0;
        maxc = max(maxc, max(a, z));
    }
    const int32_t supply = p.supply[b];
    int64_t incl = node ? max(cap, 0) : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    const int64_t total_cap = __shfl(incl, 63, 64);
    maxc = wave_max32(maxc);
    int32_t status = 0;
    if (__any(bad) || supply < 0 || total_cap > p.max_slots) status = 1;
    else if (int64_t(2 * S + 2) * maxc >= (int64_t(1) << 30)) status = 2;
    if (status == 0 && __any(cap > kMaskSlots)) {
        if (lane == 0) p.status_out[b] = kPassedOn;
        return;
    }
    int src_left = supply, sink_left = supply;
    const int my_base = int(incl) - cap;
    const uint32_t room = cap >= kMaskSlots ? ~0u : (1u << max(cap, 0)) - 1u;
    if (status == 0) {
        if (node) {
            cost[v] = cst;
            base[v] = my_base;
            usedm[v] = pairedm[v] = 0;
            for (int s = my_base; s < my_base + cap; ++s) owner[s] = uint8_t(v);
        }
        __syncthreads();
        // initial complete paths, laid out in order by lane 0
        if (p.paths && p.num_paths > 0) {
            int32_t ok = 1;
            if (lane == 0) {
                for (int q = 0; q < p.num_paths && ok; ++q) {
                    const int32_t *path = p.paths + (int64_t(b) * p.num_paths + q) * S;
                    if (path[0] < 0) continue;
                    if (src_left <= 0 || sink_left <= 0) {
                        ok = 0;
                        break;
                    }
                    int32_t prev = kData;
                    for (int kk = 0; kk < S && ok; ++kk) {
                        const int32_t j = path[kk];
                        if (j < 0 || j >= n) {
                            ok = 0;
                            break;
                        }
                        const int w = kk * n + j, cw = p.cap[int64_t(b) * V + w];
                        const uint32_t free = ~usedm[w] & (cw >= kMaskSlots ? ~0u : (1u << cw) - 1u);
                        const int32_t link = prev != kData ? lk[int(owner[prev]) * n + j] : 0;
                        if (link == kNoLink || free == 0) {
                            ok = 0;
                            break;
                        }
                        const int bit = __builtin_ctz(free), z = base[w] + bit;
                        usedm[w] |= 1u << bit;
                        pairedm[w] |= 1u << bit;
                        sin[z] = int16_t(prev);
                        slot[z] = make_int2(cost[w] + snk[j], kData);
                        if (prev != kData) slot[prev] = make_int2(cost[owner[prev]] + link, z);
                        prev = z;
                    }
                    if (ok) {
                        --src_left;
                        --sink_left;
                    }
                }
            }
            ok = __shfl(ok, 0, 64);
            src_left = __shfl(src_left, 0, 64);
            sink_left = __shfl(sink_left, 0, 64);
            if (!ok) status = 1;
            __syncthreads();
        }
    }

    double T = p.t0;
    int32_t acc = 0;
    int64_t approvals = 0;
    if (status == 0) {
        const uint64_t key0 = p.seed, key1 = uint64_t(b);
        for (int r = 0; r < p.rounds; ++r) {
            const int c = r % kChunkRounds;
            if (c == 0) {
                // ---- random numbers of the next rounds ----
                const int count = min(kChunkRounds, p.rounds - r);
                for (int it = lane; it < count * S; it += 64) {
                    // Fisher-Yates shuffle of one stage (stream 0), then every
                    // relay's partner
                    const int cc = it / S, kk = it - cc * S;
                    uint8_t *pm = perm + it * n;
                    for (int j = 0; j < n; ++j) pm[j] = uint8_t(j);
                    uint64_t words[4];
                    int block = 0;
                    for (int j = n - 1; j >= 1; j -= 4) {
                        philox(uint64_t(r + cc), uint64_t(kk), 0, uint64_t(block++), key0, key1, words);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (j - u < 1) continue;
                            const int t = draw_below(words[u], uint32_t(j - u + 1));
                            const uint8_t x = pm[j - u];
                            pm[j - u] = pm[t];
                            pm[t] = x;
                        }
                    }
                    uint16_t *to = partner + cc * V + kk * n;
                    for (int at = 0; at < n; ++at)
                        to[pm[at]] = uint16_t((at & 1) == 0 && at + 1 < n ? uint32_t(pm[at + 1]) | uint32_t(at >> 1) << 8
                                                                           : kNoPair);
                }
                for (int it = lane; it < count * S * half; it += 64) {
                    const int ck = it / half, cc = ck / S; // a pair's four draws (stream 1)
                    uint64_t w[4];
                    philox(uint64_t(r + cc), uint64_t(ck - cc * S), 1, uint64_t(it - ck * half), key0, key1, w);
                    pairs[it] = PairDraw{uint32_t(w[1] >> 32), uint32_t(w[2] >> 32), (w[3] & ~uint64_t(1)) | (w[0] & 1)};
                }
                __syncthreads();
            }
            // ---- unpaired outflow of each relay, its cost to the sink ----
            const uint32_t um = node ? usedm[v] : 0u, open = node ? um & ~pairedm[v] : 0u;
            const int32_t unp = open ? my_base + __builtin_ctz(open) : kSlotNone;
            int32_t hc = kNoHead;
            if (unp != kSlotNone) {
                hc = 0;
                int32_t s = unp;
                do {
                    const int2 w = slot[s];
                    hc += w.x;
                    s = w.y;
                } while (s != kData);
            }
            if (node) {
                head[v] = hc;
                winner[v] = kNoHead;
            }
            __syncthreads();
            // ---- Request Flow: choose targets ----
            int32_t req = kSlotNone;
            const bool wants = node && unp == kSlotNone && __popc(um) < cap;
            if (wants && k == S - 1 && sink_left > 0) req = kData;
            if (__any(unp != kSlotNone && k > 0) && wants && k < S - 1) {
                int32_t best = 0;
                for (int j = 0; j < n; ++j) {
                    const int32_t h = head[(k + 1) * n + j], l = lk[v * n + j];
                    if (h == kNoHead || l == kNoLink) continue;
                    const int32_t score = h + l;
                    if (req == kSlotNone || score < best) {
                        best = score;
                        req = (k + 1) * n + j;
                    }
                }
            }
            // approvals: lowest requester per relay target; D as sink in
            // index order while it has flow left
            const uint64_t sink_reqs = __ballot(req == kData);
            bool win = false;
            if (__any(req >= 0)) {
                if (req >= 0) atomicMin(&winner[req], v);
                __syncthreads();
                win = req >= 0 && winner[req] == v;
            }
            if (req == kData) win = wave_popc(sink_reqs & ((uint64_t(1) << v) - 1)) < sink_left;
            // D as source: first-stage unpaired outflows, cheapest first
            bool paired_by_data = false;
            if (src_left > 0 && __any(k == 0 && unp != kSlotNone)) {
                if (k == 0 && unp != kSlotNone) {
                    const int32_t mine = src[i] + hc;
                    int rank = 0;
                    for (int j = 0; j < n; ++j) {
                        if (j == i || head[j] == kNoHead) continue;
                        const int32_t other = src[j] + head[j];
                        rank += other < mine || (other == mine && j < i);
                    }
                    paired_by_data = rank < src_left;
                }
                src_left -= wave_popc(__ballot(paired_by_data));
            }
            const uint64_t wins = __ballot(win);
            if (wins) {
                sink_left -= wave_popc(__ballot(win && req == kData));
                approvals += wave_popc(wins);
            }
            if (paired_by_data) {
                sin[unp] = kData;
                pairedm[v] |= 1u << (unp - my_base);
            }
            if (win) {
                const int bit = __builtin_ctz(~um & room), z = my_base + bit;
                usedm[v] = um | 1u << bit;
                if (req == kData) {
                    slot[z] = make_int2(cst + snk[i], kData);
                } else {
                    const int ub = __builtin_ctz(usedm[req] & ~pairedm[req]), u = base[req] + ub;
                    slot[z] = make_int2(cst + lk[v * n + req - (k + 1) * n], u);
                    sin[u] = int16_t(z);
                    pairedm[req] |= 1u << ub;
                }
            }
            __syncthreads();

            // ---- improvement: even stages, then odd ones ----
            const uint32_t mate = node && req == kSlotNone ? uint32_t(partner[c * V + v]) : kNoPair;
#pragma unroll 1
            for (int parity = 0; parity < 2; ++parity) {
                if (mate != kNoPair && (k & 1) == parity) {
                    const int ib = int(mate & 255u), bn = k * n + ib;
                    const uint32_t ua = usedm[v], ub = usedm[bn], pb = pairedm[bn];
                    const bool can_redirect = __popc(ua) < cap && pb != 0;
                    const bool can_change = ua != 0 && ub != 0;
                    if (can_redirect || can_change) {
                        const PairDraw w = pairs[(c * S + k) * half + int(mate >> 8)];
                        const bool redirect = can_redirect && can_change ? (w.w3 & 1) != 0 : can_redirect;
                        const double U = double(w.w3 >> 11) * (1.0 / 9007199254740992.0);
                        const int32_t cb = cost[bn];
                        const int next0 = (k + 1) * n; // first relay of the next stage
                        // one flow of the partner's, and the other end: its
                        // inflow (redirect) or one of the proposer's flows
                        const uint32_t pick = redirect ? pb : ub;
                        const int yb = nth_bit(pick, int((uint64_t(redirect ? w.w1 : w.w2) * uint32_t(__popc(pick))) >> 32));
                        const int y = base[bn] + yb;
                        const int32_t oy = slot[y].y;
                        const int wy = oy == kData ? 0 : int(owner[oy]) - next0;
                        const int32_t c_y = oy == kData ? 0 : cost[next0 + wy];
                        const int32_t a_y = oy == kData ? snk[i] : lk[v * n + wy];
                        const int32_t b_y = oy == kData ? snk[ib] : lk[bn * n + wy];
                        int x = 0;
                        int32_t other = 0, e0, e1, n0, n1; // costs of the links given up and taken
                        bool allowed;
                        int32_t link = 0;
                        if (redirect) {
                            other = sin[y];
                            const int un = other == kData ? 0 : int(owner[other]);
                            const int32_t c_u = other == kData ? 0 : cost[un];
                            const int32_t u_a = other == kData ? src[i] : lk[un * n + i];
                            const int32_t u_b = other == kData ? src[ib] : lk[un * n + ib];
                            allowed = u_a != kNoLink && a_y != kNoLink;
                            e0 = 2 * u_b + c_u + cb;
                            e1 = 2 * b_y + cb + c_y;
                            n0 = 2 * u_a + c_u + cst;
                            n1 = 2 * a_y + cst + c_y;
                            link = c_u + u_a;
                        } else {
                            x = my_base + nth_bit(ua, int((uint64_t(w.w1) * uint32_t(__popc(ua))) >> 32));
                            other = slot[x].y;
                            const int wx = other == kData ? 0 : int(owner[other]) - next0;
                            const int32_t c_x = other == kData ? 0 : cost[next0 + wx];
                            const int32_t a_x = other == kData ? snk[i] : lk[v * n + wx];
                            const int32_t b_x = other == kData ? snk[ib] : lk[bn * n + wx];
                            const bool same = (other == kData) == (oy == kData) && wx == wy;
                            allowed = !same && a_y != kNoLink && b_x != kNoLink;
                            e0 = 2 * a_x + cst + c_x;
                            e1 = 2 * b_y + cb + c_y;
                            n0 = 2 * a_y + cst + c_y;
                            n1 = 2 * b_x + cb + c_x;
                            link = cb + b_x;
                        }
                        const int32_t cur = p.objective ? max(e0, e1) : e0 + e1;
                        const int32_t nxt = p.objective ? max(n0, n1) : n0 + n1;
                        if (allowed && accepts(cur, nxt, T, U)) {
                            T *= p.alpha;
                            ++acc;
                            if (redirect) {
                                const int bit = __builtin_ctz(~ua & room);
                                x = my_base + bit;
                                usedm[v] = ua | 1u << bit;
                                pairedm[v] |= 1u << bit;
                                usedm[bn] = ub & ~(1u << yb);
                                pairedm[bn] = pb & ~(1u << yb);
                                sin[x] = int16_t(other);
                                if (other != kData) slot[other] = make_int2(link, x);
                            } else {
                                slot[y] = make_int2(link, other);
                                if (other != kData) sin[other] = int16_t(y);
                            }
                            slot[x] = make_int2(cst + a_y, oy);
                            if (oy != kData) sin[oy] = int16_t(x);
                        }
                    }
                }
                __syncthreads();
            }
        }
    }

    // ---- result: complete paths, stage by stage from the source ----
    int32_t nf = 0, used = 0;
    int64_t mycost = 0;
    uint32_t done = 0; // slots of this relay on complete paths
    uint32_t *donem = reinterpret_cast<uint32_t *>(head);
    if (status == 0) {
        for (int kk = 0; kk < S; ++kk) {
            if (node && k == kk) {
                used = __popc(usedm[v]);
                for (uint32_t m = pairedm[v]; m; m &= m - 1) {
                    const int bit = __builtin_ctz(m), s = my_base + bit;
                    const int32_t in = sin[s];
                    const int w = in >= 0 ? int(owner[in]) : 0;
                    if (in == kData || ((donem[w] >> (in - base[w])) & 1u)) {
                        done |= 1u << bit;
                        mycost += slot[s].x + (k == 0 ? src[i] : 0);
                    }
                }
                nf = __popc(done);
                donem[v] = done;
            }
            __syncthreads();
        }
    }
    const int64_t F = wave_sum64(node && k == 0 ? nf : 0);
    const int64_t total = wave_sum64(mycost);
    const int64_t accepted = wave_sum64(acc);
    const int64_t dangling = wave_sum64(used - nf);
    if (lane == 0) {
        p.F_out[b] = status == 0 ? F : 0;
        p.cost_out[b] = status == 0 ? total : 0;
        p.status_out[b] = status;
        if (p.counters) {
            int64_t *to = p.counters + int64_t(b) * 4;
            to[0] = status == 0 ? supply - src_left : 0;
            to[1] = status == 0 ? approvals : 0;
            to[2] = status == 0 ? accepted : 0;
            to[3] = status == 0 ? dangling : 0;
        }
    }
    if (node) {
        const int64_t at = int64_t(b) * V + v;
        if (p.node_flow) p.node_flow[at] = nf;
        if (p.used) p.used[at] = used;
        if (p.accepted) p.accepted[at] = acc;
        if (p.temperature) p.temperature[at] = T;
        if (p.arc_flow && k < S - 1) {
            int32_t *row = p.arc_flow + (int64_t(b) * (S - 1) + k) * n * n + int64_t(i) * n;
            for (int j = 0; j < n; ++j) row[j] = 0;
            for (uint32_t m = done; m; m &= m - 1)
                row[int(owner[slot[my_base + __builtin_ctz(m)].y]) - (k + 1) * n] += 1;
        }
    }
}

} // namespace

size_t heuristic_lds_bytes(int S, int n, int max_slots)
{
    const size_t general = heur_layout(S, n, max_slots).total;
    const size_t masks = mask_layout(S, n, max_slots).total;
    return general > masks ? general : masks;
}

hipError_t launch_heuristic(const HeurParams &p, const LaunchInfo &l, hipStream_t stream)
{
    const size_t fast = mask_layout(p.S, p.n, p.max_slots).total, general = heur_layout(p.S, p.n, p.max_slots).total;
    for (auto [f, bytes] : {std::pair{reinterpret_cast<const void *>(heuristic_kernel), fast},
                            std::pair{reinterpret_cast<const void *>(heuristic_general_kernel), general}})
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess)
            (void)hipGetLastError();
    hipLaunchKernelGGL(heuristic_kernel, dim3(unsigned(p.B)), dim3(64), fast, stream, p);
    const hipError_t e = hipGetLastError();
    // The second launch costs 4 us where it finds nothing to do (one instance of
    // 8 x 5: one round 31 us before there were two forms, 36 now; 120 rounds 2,154
    // and 416).
    if (e != hipSuccess || p.max_slots <= kMaskSlots || l.first_only) return e; // no relay can hold more
    hipLaunchKernelGGL(heuristic_general_kernel, dim3(unsigned(p.B)), dim3(64), general, stream, p);
    return hipGetLastError();
}

} // namespace gwtf
