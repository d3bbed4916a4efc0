// Packed pass for small instances: one to sixteen instances per wave, for at
// most 16 stages of at most 16 nodes (the node-addition batches of paper
// Sec. VI, its flow tests and the 4 x 4 / 8 x 8 presets).
//
// Same method as the other passes (successive shortest paths with Johnson
// potentials on the node-split stage graph, paper Sec. V-A Eq. 2); what
// differs is the mapping.  A wave is cut into groups of G = 4, 8 or 16 lanes
// (the smallest that holds a stage), one instance per group, lane j of a
// group = node j of every stage; a small batch leaves some groups of each
// wave empty so that it spreads over more waves:
//
//  * Keys.  A vertex label is kept as key = label << 5 | code, where code
//    names the predecessor arc: for an entry, 0..15 = the link from that
//    exit of the previous stage, 16 = the reverse compute arc, 17 = the
//    data node; for an exit, 0..15 = the reverse link from that entry of the
//    next stage, 16 = the compute arc.  Finite keys stay below 2^30 (labels
//    below 2^25); unreached vertices hold 2^30 | 31, a missing link costs
//    2^30, and an unreached label that a cost is subtracted from counts as
//    2^31, so no candidate that involves an unreached vertex or a missing
//    link lands in the finite range and nothing wraps.  A key is replaced
//    only by one with a strictly smaller label, which keeps the predecessors
//    a tree.
//  * Forward relaxation.  The incoming link costs of a stage sit in vector
//    registers (cost << 5, column j in lane j).  For G = 16 exit i's key
//    reaches every lane through a DPP row broadcast fused into the add, for
//    the first ROWS = 10, 13 or 16 exits.  For
//    G = 4 and 8 the lanes exchange keys by XOR: register d of lane j holds
//    the cost of the link from exit j ^ d, and the quad permutes (with one
//    half-row mirror for d >= 4) deliver lane j ^ d's key inside the add, so
//    a dense 8 x 8 relaxation is 9 instructions and 4 three-way minima
//    (two bank-masked broadcasts per row and an add before: 28).
//  * Reverse links (links carrying flow) are pulled at the exit's lane from
//    the next stage's entry keys.  For G = 4 and 8 the costs of all of an
//    exit's links sit in registers too, kOff below their value while the link
//    carries no flow (its candidate then lies above the finite range), so a
//    pull is the same exchange with subtractions; they are reloaded from
//    their LDS copy before each search.  For G = 16 (no registers left) the
//    exit's set bits of a 16-bit mask are taken two per pass.
//  * Rounds: a forward sweep over the stages, then a backward sweep; stages
//    whose input has not changed are skipped.  A search is over when
//    a backward sweep changes no exit key in any of the wave's instances.
//    (Letting groups that converged early augment and start their next
//    search while the others go on was slower: 562 us against 664 with three
//    and 904 with one waiting group on 16,384 instances of 8 x 8, since the
//    augmentation then runs for few groups at a time.)
//  * After each search: potentials (registers), then each group walks its
//    path over a table of the nodes' predecessor codes in LDS, one read per
//    node, and lists the nodes it meets; lane s of the group then takes the
//    s-th of them, for the bottleneck and again to apply the path, so that a
//    path costs two short steps and not two passes over all stages.  The
//    table carries the node flows too; the lanes take theirs back from it.
//
// What bounds it: the chain of dependent instructions of a stage step (about
// 21 vector instructions, eight cycles each for a wave that has its SIMD to
// itself) and, with two waves per SIMD, instruction issue; HBM traffic is the
// inputs and the flow export.  Measured against the form with row broadcasts,
// node words read from LDS in every step and a recorded path (before / now):
// 16,384 of 8 x 8 1,418 / 461 us, 1,024 of 4 x 4 135 / 59, one 8 x 8 494 /
// 191, 40,320 of 8 x 13 with expansion 8.7 / 4.9 ms; 11,880 of 12 x 9 on one
// wave per instance 27.5, here 3.4 ms with expansion.
//
// The first launch takes instances with supply <= 255 and costs <= 2047
// (link flows in 8 bits).  The second (solve_small_rest_kernel) takes what
// that one passed on, in the same way with 16-bit flows while labels stay
// below 2^25 and the value below 2^16, and one instance per wave by the
// general method (mcf_solve_body.h) beyond that, in a third launch for large
// batches of more than 8 stages (launch_stages); its workgroups leave at once
// when there is nothing to do (5 us for 16,384 instances).  A workgroup of 16
// waves per instance with its state in device memory took 42.0 ms for 4,096
// instances of 8 x 5 with supplies above 255 (now 0.37) and 26.8 ms for 1,500
// of 7 x 11 with costs up to 6000 (now 0.77).
#pragma once

#include "mcf_small_device.h"
#include "mcf_solve_body.h"
#include "mcf_small.h"

#include <algorithm>
#include <type_traits>

namespace gwtf {
namespace {

using namespace dev;

template <bool WIDE> struct FlowType { using type = uint8_t; };
template <> struct FlowType<true> { using type = uint16_t; };
template <bool WIDE> struct CostType { using type = uint16_t; };
template <> struct CostType<true> { using type = uint32_t; };

// Solves instances blockIdx.x * R ... + R - 1 (those the first launch passed
// on when WIDE).  Writes `route` for each instance it finishes and leaves
// kRouteFallback for the others; true in the lanes of
// the groups it left.
template <int MAXS, int G, int ROWS, bool WIDE>
__device__ __forceinline__ bool solve_rows(const SolveParams &p, int R, int32_t route_done, unsigned char *smem)
{
    using Flow = typename FlowType<WIDE>::type;
    using Cost = typename CostType<WIDE>::type;
    constexpr bool XOR = G < 16;
    constexpr int kMaxCost = max_cost(WIDE), kMaxSupply = max_supply(WIDE);
    GWTF_PHASE;
    const int SN = S * n, V = 2 * SN + 3;
    const int b = blockIdx.x * R + g;
    const bool inst = g < R && b < p.B && (!WIDE || p.route[b] == kRouteFallback);
    const bool node = inst && j < n; // this lane is a real node
    const SmallLayout Ly = small_layout<MAXS, G, WIDE>(S, n, R);
    using W = Word<WIDE>;
    using Path = typename PathType<MAXS * G <= 128>::type;
    typename W::type *table = reinterpret_cast<typename W::type *>(smem); // [S][64]
    Path *path = reinterpret_cast<Path *>(smem + Ly.path);             // [R][kPathChunk]
    Flow *lflow = reinterpret_cast<Flow *>(smem + Ly.flow);            // [S-1][R][n][n]: (k, i) -> (k+1, j)
    Cost *lcost = reinterpret_cast<Cost *>(smem + Ly.cost);            // [S-1][R][n][n], G = 16
    uint32_t *rcost = reinterpret_cast<uint32_t *>(smem + Ly.cost);    // [S-1][R * G][G], G < 16
    uint32_t *lmask = reinterpret_cast<uint32_t *>(smem + Ly.mask);    // [S-1][64], G = 16
    const int supply = inst ? p.supply[b] : 0;
    const int32_t *gcap = p.cap + size_t(b) * SN;
    const int32_t *gnc = p.ncost + size_t(b) * SN;
    const int32_t *gac = S > 1 ? p.acost + size_t(b) * (S - 1) * nn : nullptr;

    auto flow_of = [](typename W::type w) GWTF_INLINE { return uint32_t(w >> W::flow) & W::mask; };
    auto cap_of = [](typename W::type w) GWTF_INLINE { return uint32_t(w >> W::cap) & W::mask; };

    // ---------------- ingest + validate ----------------
    int bad = supply < 0, mx = 0;
    uint32_t cin[MAXS][ROWS];             // cost << 5 of the links into node (k, j), k >= 1: from exit d (XOR: j ^ d)
    typename W::type nw[MAXS];         // the node's flow and capacity, as in its table word
    uint32_t nc5[MAXS];                // its compute cost << 5
    uint32_t value = uint32_t(max(supply, 0)); // bound on the flow value: the supply and every stage's capacity
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        nw[k] = 0;
        nc5[k] = 0;
        if (k >= S) return;
        const int cp = node ? gcap[k * n + j] : 0, w = node ? gnc[k * n + j] : 0;
        bad |= (cp < 0) | (w < 0);
        mx = max(mx, w);
        value = min(value, group_sum<G>(uint32_t(min(max(cp, 0), 1 << 20))));
        nw[k] = typename W::type(min(min(max(cp, 0), max(supply, 0)), kMaxSupply)) << W::cap;
        nc5[k] = uint32_t(min(max(w, 0), kMaxCost)) << 5;
    });
    each<MAXS - 1, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k + 1 >= S) return;
        int a[ROWS];
#pragma unroll
        for (int d = 0; d < ROWS; ++d) {
            // XOR: the links out of node j; G = 16: the links into it
            const int i = XOR ? j : d, jj = XOR ? j ^ d : j;
            a[d] = (node && i < n && jj < n) ? gac[k * nn + i * n + jj] : -1;
        }
#pragma unroll
        for (int d = 0; d < ROWS; ++d) {
            bad |= a[d] < -1;
            mx = max(mx, a[d]);
            const bool hole = a[d] < 0;
            const uint32_t c5 = uint32_t(min(max(a[d], 0), kMaxCost)) << 5;
            if constexpr (XOR) {
                if (g < R) rcost[ridx(k, lane, d)] = c5 - kOff;
                // missing links and padding: never a candidate
                cin[k + 1][d] = hole ? kNoLink : c5;
            } else {
                // an instance's own rows only; padding rows hold no link
                cin[k + 1][d] = hole ? kNoLink : c5;
                if (g < R && d < n && j < n) lcost[lidx(k, d, j)] = Cost(c5);
            }
        }
        if constexpr (XOR) {
            // the links into node j: register d from the row of node j ^ d
            turn<G>(cin[k + 1]);
        } else {
            lmask[k * 64 + lane] = 0;
        }
        if (g < R)
            for (int e = j; e < nn; e += G) lflow[(k * R + g) * nn + e] = 0;
    });
    const int srcc = node && p.src ? p.src[size_t(b) * n + j] : 0;
    const int snkc = node && p.snk ? p.snk[size_t(b) * n + j] : 0;
    bad |= (srcc < 0) | (snkc < 0);
    mx = max(mx, max(srcc, snkc));
    bad = group_max<G>(bad);
    mx = group_max<G>(mx);
    int status = 0;
    if (bad) status = 1;
    else if (int64_t(V) * mx >= kLabelBound) status = 2;
    const bool fits = (WIDE ? value <= uint32_t(kMaxSupply) : supply <= kMaxSupply) && mx <= kMaxCost &&
                      int64_t(V) * mx < kSmallLabelLimit;
    const bool mine = inst && (status != 0 || fits); // this form owns the instance
    if (inst && j == 0) p.route[b] = mine ? route_done : kRouteFallback;
    const uint32_t src5 = uint32_t(min(max(srcc, 0), kMaxCost)) << 5, snk5 = uint32_t(min(max(snkc, 0), kMaxCost)) << 5;
    __syncthreads();

    // ---------------- successive shortest paths ----------------
    const int goal = int(value); // no flow has a larger value
    int F = 0, augs = 0, rounds = 0;
    long long cost = 0, rows_relaxed = 0;
    // reverse-link relaxations of this lane: at most 65,535 searches of 259
    // rounds over 15 * 8 links for G < 16
    std::conditional_t<XOR, uint32_t, uint64_t> pulls = 0;
    uint32_t pit = 0; // the sink's potential, << 5 as all labels here
    bool active = mine && status == 0 && goal > 0; // this group still searches
    uint64_t tick = wall_clock64(), clk_label = 0, clk_aug = 0;
    uint32_t din[MAXS], dout[MAXS], ncf[MAXS], ncr[MAXS];
    // Potentials of this lane's entries and exits, less the sink's: after
    // each search min(label - the sink's label, what it was).
    int32_t pin[MAXS], pout[MAXS];
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        pin[k] = pout[k] = 0;
    });
    while (__any(active)) {
        // XOR: the costs of the links out of exit (k, j) to node j ^ d, as in LDS
        uint32_t rc[XOR ? MAXS : 1][G];
        {
            GWTF_PHASE;
            // labels of a fresh search, and the residual compute arcs: forward
            // while the node has room, backward (code 16 folded in) while it
            // carries flow
            each<MAXS, false>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                din[k] = dout[k] = kKeyInf;
                if (k == 0 && active && j < n) din[k] = src5 | kCodeSrc;
                if (k >= S) return;
                const uint32_t fl = flow_of(nw[k]), ec = cap_of(nw[k]);
                ncf[k] = fl < ec ? nc5[k] + kCodeSplit : kNoLink;
                ncr[k] = (fl > 0 ? nc5[k] : nc5[k] - kOff) - kCodeSplit;
                if constexpr (XOR) {
                    if (k + 1 < S) {
#pragma unroll
                        for (int d = 0; d < G; ++d) rc[k][d] = rcost[ridx(k, g < R ? int(lane) : j, d)];
                    }
                }
            });
        }
        const bool flowing = __any(F > 0);
        int round_count = 0;
        bool fault = false;
        // Stages whose exit (entry) keys changed in some lane since the next
        // (previous) stage last read them: a relaxation or a pull whose input
        // is unchanged cannot improve anything and is skipped, and with it
        // the stage's compute arcs (a label they could improve changed only
        // through that relaxation or pull).  Bit kBegin: a new search.
        constexpr uint32_t kBegin = 1u << 31;
        uint32_t new_out = kBegin;
        for (;;) {
            GWTF_PHASE;
            const uint32_t last = 1u << (S - 1);
            // -------- forward sweep --------
            uint32_t new_in = 0;
            each<MAXS, false>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                if constexpr (k == 0) {
                    if (!(new_out & kBegin)) return;
                } else {
                    if (!(new_out & (1u << (k - 1)))) return;
                    const uint32_t best = exchange<G, false, ROWS>(label_of(dout[k - 1]) | uint32_t(j), cin[k]);
                    const bool better = best < label_of(din[k]);
                    rows_relaxed += n;
                    if (!__any(better)) return;
                    din[k] = better ? best : din[k];
                    new_in |= 1u << k;
                }
                const uint32_t cand = label_of(din[k]) + ncf[k];
                const bool take = cand < label_of(dout[k]);
                dout[k] = take ? cand : dout[k];
                if (__any(take)) new_out |= (1u << k) & (last - 1);
            });
            new_out = 0;
            // -------- backward sweep --------
            if (flowing) {
                each<MAXS - 1, true>([&](auto K) GWTF_INLINE {
                    constexpr int k = K;
                    if (!(new_in & (2u << k))) return;
                    const uint32_t yr = sub_tail(label_of(din[k + 1])) | uint32_t(j);
                    uint32_t best;
                    if constexpr (XOR) {
                        best = exchange<G, true, G>(yr, rc[k]);
                        // links with flow out of the exit: its word's top four
                        // bits, in one instruction
                        pulls = __builtin_amdgcn_udot8(uint32_t(nw[k]), 1u << kLinksAt, pulls, false);
                    } else {
                        // links with flow out of this exit, two per pass
                        uint32_t rem = lmask[k * 64 + lane];
                        best = ~0u;
                        pulls += __popc(rem);
                        while (__any(rem != 0u)) {
                            const bool h0 = rem != 0u;
                            const int j0 = h0 ? __builtin_ctz(rem) : 0;
                            rem &= rem - 1u;
                            const bool h1 = rem != 0u;
                            const int j1 = h1 ? __builtin_ctz(rem) : 0;
                            rem &= rem - 1u;
                            const uint32_t y0 = uint32_t(__shfl(int(yr), gb + j0)), y1 = uint32_t(__shfl(int(yr), gb + j1));
                            // only a real exit with a partner reads its cost
                            const uint32_t c0 = h0 ? uint32_t(lcost[lidx(k, j, j0)]) : 0u;
                            const uint32_t c1 = h1 ? uint32_t(lcost[lidx(k, j, j1)]) : 0u;
                            best = h0 ? min(best, y0 - c0) : best;
                            best = h1 ? min(best, y1 - c1) : best;
                        }
                    }
                    const bool take = best < label_of(dout[k]);
                    if (!__any(take)) return;
                    dout[k] = take ? best : dout[k];
                    new_out |= 1u << k;
                    const uint32_t cand = sub_tail(label_of(dout[k])) - ncr[k];
                    const bool tin = cand < label_of(din[k]);
                    din[k] = tin ? cand : din[k];
                    if (__any(tin)) new_in |= 1u << k;
                });
            }
            ++rounds;
            if (new_out == 0) break; // the backward sweep changed no exit, so no entry either
            // Bellman-Ford settles within |V| rounds without a negative cycle
            if (++round_count > V) {
                fault = true;
                break;
            }
        }
        clk_label += lap(tick);
        if (fault) {
            if (active) status = kStatusInternal;
            break;
        }

        // -------- sink, potentials --------
        GWTF_PHASE;
        uint32_t tk = kKeyInf;
        each<MAXS, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k == S - 1) tk = dout[k];
        });
        tk = group_min<G>(j < n ? (label_of(tk) + snk5) | uint32_t(j) : kKeyInf);
        const bool aug = active && tk < kFinite;
        active = aug; // sink unreachable: the flow is maximum
        const uint32_t Dt = label_of(tk); // << 5
        const int32_t less = aug ? int32_t(Dt) : 1 - int32_t(kFinite); // a group that stops here keeps its potentials
        each<MAXS, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k >= S) return;
            pin[k] = min(pin[k], int32_t(label_of(din[k])) - less);
            pout[k] = min(pout[k], int32_t(label_of(dout[k])) - less);
            table[k * 64 + lane] = ((dout[k] << 5) & 0x3e0u) | ((din[k] & 31u) | nw[k]);
        });
        wave_sync();

        // -------- path: list its nodes, bottleneck, then apply --------
        // Walk: one table read per node.  An exit reached by its compute arc
        // goes on from the entry's code in the same step.
        bool bad_walk = false, open = false; // open: the path goes on beyond the listed nodes
        int wk = 0, wv = 0, listed = 0, total = 0;
        bool at_exit = true;
        auto walk_begin = [&]() GWTF_INLINE {
            wk = S - 1;
            wv = int(tk & 31u);
            at_exit = open = aug;
            total = 0;
        };
        auto walk = [&]() GWTF_INLINE {
            listed = 0;
            bool go = open;
            while (go) {
                const uint32_t w = uint32_t(table[wk * 64 + gb + wv]);
                const uint32_t ce = (w >> 5) & 31u, ci = w & 31u;
                path[g * kPathChunk + listed] = Path(((wk * G + wv) << 1) | int(at_exit));
                ++listed;
                const bool via = at_exit && ce != kCodeSplit; // leaves by a reverse link
                const uint32_t code = via ? ce : ci;
                const bool back = code == kCodeSplit;         // reverse compute arc: on to the own exit
                open = via || code != kCodeSrc;
                wk += via ? 1 : (back ? 0 : -1);
                wv = back ? wv : int(code & 15u);
                at_exit = !via;
                if (open && (code > kCodeSplit || uint32_t(wk) >= uint32_t(S))) {
                    bad_walk = true;
                    open = false;
                }
                go = open && listed < kPathChunk;
            }
            total += listed;
            if (total > 2 * S * G + 4) { // longer than the vertex count
                bad_walk = true;
                open = false;
            }
        };
        // f(table index of the node, entry part, exit part leaves by a
        // reverse link, exit part is its compute arc, entry code, link index
        // and tail (stage, node), head node) of the listed node of this lane
        auto each_listed = [&](auto f) GWTF_INLINE {
            for (int at = j; __any(at < listed); at += G) {
                if (at < listed) {
                    const int rec = int(path[g * kPathChunk + at]), k = (rec >> 1) / G, v = (rec >> 1) % G;
                    const int q = k * 64 + gb + v;
                    const typename W::type w = table[q];
                    const uint32_t ce = uint32_t(w >> 5) & 31u, ci = uint32_t(w) & 31u;
                    const bool ex = (rec & 1) != 0, via = ex && ce != kCodeSplit;
                    const bool link = via || ci < 16;
                    const int lk = via ? k : k - 1, tail = via ? v : int(ci), head = via ? int(ce) : v;
                    f(q, w, via, ex && !via, !via && ci == kCodeSplit, link, lk, tail, head);
                }
            }
        };
        uint32_t room = aug ? uint32_t(goal - F) : 0u;
        int chunks = 0;
        walk_begin();
        do {
            walk();
            wave_sync();
            each_listed([&](int, typename W::type w, bool via, bool split, bool back, bool, int lk, int tail,
                            int head) GWTF_INLINE {
                if (split) room = min(room, cap_of(w) - flow_of(w));
                if (back) room = min(room, flow_of(w));
                if (via) room = min(room, uint32_t(lflow[lidx(lk, tail, head)]));
            });
            ++chunks;
        } while (__any(open));
        const uint32_t delta = group_min<G>(room);
        if (aug && int(delta) <= 0) bad_walk = true;
        if (bad_walk) {
            status = kStatusInternal;
            active = false;
        }
        const bool apply = aug && !bad_walk;
        if (chunks > 1) walk_begin();
        do {
            if (chunks > 1) {
                wave_sync();
                walk();
                wave_sync();
            }
            if (!apply) listed = 0;
            // a simple path holds each compute arc and each link once
            each_listed([&](int q, typename W::type, bool via, bool split, bool back, bool link, int lk, int tail,
                            int head) GWTF_INLINE {
                uint32_t *flow_word = reinterpret_cast<uint32_t *>(&table[q]);
                if (split) atomicAdd(flow_word, delta << W::flow);
                if (back) atomicSub(flow_word, delta << W::flow);
                if (link) {
                    const int e = lidx(lk, tail, head);
                    const uint32_t had = uint32_t(lflow[e]);
                    lflow[e] = Flow(via ? had - delta : had + delta);
                    if (had == (via ? delta : 0u)) { // the link empties or begins to carry flow
                        if constexpr (XOR) {
                            atomicAdd(&rcost[ridx(lk, gb + tail, tail ^ head)], via ? 0u - kOff : kOff);
                            atomicAdd(reinterpret_cast<uint32_t *>(&table[lk * 64 + gb + tail]),
                                      via ? 0u - (1u << kLinksAt) : 1u << kLinksAt);
                        } else {
                            uint32_t *mask = &lmask[lk * 64 + gb + tail];
                            if (via) atomicAnd(mask, ~(1u << head));
                            else atomicOr(mask, 1u << head);
                        }
                    }
                }
            });
        } while (chunks > 1 && __any(open));
        wave_sync();
        each<MAXS, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k >= S) return;
            nw[k] = table[k * 64 + lane] & ~typename W::type(1023);
        });
        if (apply) {
            F += int(delta);
            cost += (long long)delta * (long long)(Dt >> 5);
            ++augs;
            pit = Dt;
            if (F >= goal) active = false;
        }
        clk_aug += lap(tick);
    }

    // ---------------- export ----------------
    uint64_t all_pulls = pulls;
    for (int o = G / 2; o > 0; o >>= 1) all_pulls += __shfl_xor(all_pulls, o);
    if (mine) {
        const bool ok = status == 0;
        const size_t na = size_t(S > 1 ? S - 1 : 0) * nn;
        int32_t *nf = p.node_flow + size_t(b) * SN;
        int32_t *af = p.arc_flow + size_t(b) * na;
        int32_t *gpot = p.pot + size_t(b) * V;
        each<MAXS, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k >= S) return;
            if (j < n) {
                const int q = k * n + j;
                nf[q] = ok ? int(flow_of(nw[k])) : 0;
                gpot[3 + 2 * q] = ok ? (pin[k] + int32_t(pit)) >> 5 : 0;
                gpot[4 + 2 * q] = ok ? (pout[k] + int32_t(pit)) >> 5 : 0;
            }
            if (k + 1 < S)
                for (int e = j; e < nn; e += G) af[size_t(k) * nn + e] = ok ? int(lflow[(k * R + g) * nn + e]) : 0;
        });
        if (j == 0) {
            gpot[0] = 0;
            gpot[1] = 0;
            gpot[2] = ok ? int(pit >> 5) : 0;
            p.F_out[b] = ok ? F : 0;
            p.cost_out[b] = ok ? cost : 0;
            p.status_out[b] = status;
            int64_t *s = p.stats + size_t(b) * kStatsPerInstance;
            s[0] = augs;
            s[1] = rounds;
            s[2] = rows_relaxed;
            s[3] = int64_t(all_pulls);
            const double ns_per_tick = 1e6 / double(p.clock_khz > 0 ? p.clock_khz : 100000);
            s[4] = int64_t(double(clk_label) * ns_per_tick); // both sweeps
            s[5] = 0;
            s[6] = int64_t(double(clk_aug) * ns_per_tick);
            s[7] = 0;
            s[8] = 0;
            s[9] = 0;
        }
    }
    return inst && !mine;
}

template <int MAXS, int G, int ROWS>
__global__ __launch_bounds__(64, MAXS > 8 ? 1 : 2) void solve_small_kernel(SolveParams p, int R, int32_t route_done)
{
    extern __shared__ __align__(16) unsigned char smem[];
    solve_rows<MAXS, G, ROWS, false>(p, R, route_done, smem);
}

// Instances the first launch passed on: R at a time with wide values, then,
// when `general`, what is left one after another.
template <int MAXS, int G, int ROWS>
__global__ __launch_bounds__(64, MAXS > 8 ? 1 : 2) void solve_small_rest_kernel(SolveParams p, int R, int32_t route_done,
                                                                                 bool general)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int first = blockIdx.x * R, lane = threadIdx.x;
    if (!__any(lane < R && first + lane < p.B && p.route[first + lane] == kRouteFallback)) return;
    uint64_t left = __ballot(solve_rows<MAXS, G, ROWS, true>(p, R, route_done, smem) && lane % G == 0);
    while (general && left) {
        const int r = __builtin_ctzll(left) / G;
        left &= left - 1;
        __syncthreads();
        solve_body<1, true>(p, first + r, route_done, smem);
    }
}

template <int MAXS, int G, int ROWS> hipError_t launch_stages(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    const int S = p.S, n = p.n;
    const int R = rows_per_wave(64 / G, p.B, l.cus);
    const size_t lds = small_layout<MAXS, G, false>(S, n, R).total;
    if (lds > l.lds_max) return hipErrorInvalidValue;
    hipLaunchKernelGGL((solve_small_kernel<MAXS, G, ROWS>), dim3(unsigned((p.B + R - 1) / R)), dim3(64), lds, s, p, R,
                       S <= kPackedStages ? kRouteSmall : kRouteLds);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || l.first_only) return e;
    // The rest: what it holds per wave is bounded by 40 KB of LDS.
    int Rr = R;
    while (Rr > 1 && small_layout<MAXS, G, true>(S, n, Rr).total > 40 * 1024) Rr /= 2;
    SolveParams q = p;
    q.list_slots = int64_t(S > 1 ? S - 1 : 0) * n * n; // lists of the worst case: at most 3840 entries
    const size_t body = make_layout(S, n, q.list_slots, true).total + scratch_bytes(1, n);
    // With more than 8 stages the rest kernel's registers let one wave run per
    // SIMD, a lean workgroup's let as many as its LDS allows: what the wide form
    // leaves goes to a launch of its own once a wave would hold several of them
    // (costs around half a million, 16,384 instances of 9 x 4: 13.1 ms within
    // the rest launch, 4.1 in their own; 4,096 of 12 x 9: 35.0 and 15.4; 16,384 of
    // 16 x 4: 27.0 and 8.4).  Where it finds nothing to do that launch costs 2 us
    // for 4,096 instances and 5 for 16,384.
    // One instance per wave takes as long in either (12 x 9: 3.8 ms alone, 9.4
    // for 256), and with at most 8 stages the rest launch is the faster way than
    // the fallback pass's workgroup of 16 waves (one 8 x 8 1.7 against 2.6 ms,
    // 16,384 of them 41 against 242 ms).
    const bool general = S <= kPackedStages || R == 1;
    const size_t rows = small_layout<MAXS, G, true>(S, n, Rr).total, rest = general ? std::max(rows, body) : rows;
    if (rows > l.lds_max || body > l.lds_max) return hipErrorInvalidValue;
    hipLaunchKernelGGL((solve_small_rest_kernel<MAXS, G, ROWS>), dim3(unsigned((p.B + Rr - 1) / Rr)), dim3(64), rest, s, q,
                       Rr, S <= kPackedStages ? kRouteGlobal : kRouteLds, general);
    if ((e = hipGetLastError()) != hipSuccess || general) return e;
    return launch_lds_pass(q, 1, body, s);
}

template <int G, int ROWS> hipError_t launch_group(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    return p.S <= kPackedStages ? launch_stages<kPackedStages, G, ROWS>(p, l, s)
                                : launch_stages<kSmallMaxStages, G, ROWS>(p, l, s);
}

} // namespace
} // namespace gwtf
