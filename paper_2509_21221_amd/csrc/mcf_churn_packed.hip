// Packed form of the warm-started churn re-solve (mcf_churn.hip has the method
// and the general form): several instances per wave for S <= 8, n <= 16, with
// the lane mapping, keys and exchanges of the packed pass (mcf_small_kernel.h).
//
// What differs from the cold solve there:
//  * Start.  The start flow's links go to LDS, its node flows to the walk
//    table; each group strips paths as the general form does, the lanes of the
//    group looking for the next link with flow together.
//  * Negative cycles may pass through the data node, so its two sides s and t
//    have keys of their own, the same in every lane of a group.  The arcs
//    between s and stage 0 (stage S-1 and t) carry exactly the flow of the
//    nodes there and need no flow words.
//  * In the cancelling phase all labels start at 0, kept as kZero so that keys
//    stay positive: a round lowers a label by at most the 2 (2 S + 2) arcs a
//    forward and a backward sweep can chain, so kRoundCap rounds of costs up to
//    2047 take less than 2^24 off it.  Predecessors of a label that never
//    changed end in code 31.
//  * After every second round a group that still cancels follows the
//    predecessors of an exit that the round's backward sweep changed (Brent's
//    cycle finding, one table read per node).  Changes that do not come from a
//    negative cycle die out, so sooner or later that exit lies behind one.  The
//    group lists the cycle's nodes, takes its labels out of the search and
//    waits for the others; cycles and augmenting paths are then pushed
//    together, one lane per listed node.  (On the variants below: 1.52 ms with
//    a check after each round, 1.42 from the second round on, 1.33 from the
//    third, 1.29 after every second.)
//  * Groups of one wave are in different phases; only labels differ.
//
// Whatever this form does not hold (supply, start flows above 255, costs above
// 2047, invalid input, a path or cycle of more than 64 listed nodes) is marked
// kChurnPassedOn in the instance's status and solved by the general form,
// launched right after.  An instance passed on for its values pays for this
// launch's ingest: costs above 2047, one 8 x 8 2.00 -> 2.02 ms, 4,096 3.57 ->
// 3.58 ms.
//
// What bounds it: the dependent instructions of a search, as in the packed
// pass, for about 20 searches per variant instead of its 17; a lone lane's
// walks and one instance per wave bounded the general form.  16,384 variants
// of 8 x 8: 8.7 ms there, 1.29 ms here (75 rounds per variant; 285 there).
#include "gwtf_mcf.h"
#include "mcf_churn.h"
#include "mcf_small_device.h"

namespace gwtf {
namespace {

using namespace dev;

constexpr uint32_t kZero = 0x20000000u; // label 0
// Rounds of one search: 36 arcs * 2047 * 200 < 2^24.  No search gets there.  A
// label that changed in round r has a predecessor that changed in the same round,
// or in the round before it when the sweep turns, so a chain of predecessors that
// ends in a root has 2 r vertices or more; with at most 258 vertices a label that
// still changes after 130 rounds lies behind a cycle, which the next check finds.
constexpr int kRoundCap = 200;
constexpr int kTotalRounds = 1 << 20;   // of all cancelling searches; the general form restarts from zero there
constexpr uint32_t kRoot = 31;          // code of a label without predecessor
constexpr uint32_t kUnbounded = 1u << 20;

template <int G> __global__ __launch_bounds__(64, 2) void churn_packed_kernel(ChurnParams p, int R)
{
    constexpr int MAXS = kChurnPackedStages;
    constexpr bool XOR = G < 16;
    using W = Word<false>;
    extern __shared__ __align__(16) unsigned char smem[];
    GWTF_PHASE;
    const int SN = S * n, V = 2 * SN + 2;
    const int b = blockIdx.x * R + g;
    const bool inst = g < R && b < p.B;
    const bool node = inst && j < n;
    const SmallLayout Ly = small_layout<MAXS, G, false>(S, n, R);
    uint32_t *table = reinterpret_cast<uint32_t *>(smem);             // [S][64]
    uint8_t *path = smem + Ly.path;                                   // [R][kPathChunk]
    uint8_t *lflow = smem + Ly.flow;                                  // [S-1][R][n][n]
    uint16_t *lcost = reinterpret_cast<uint16_t *>(smem + Ly.cost);   // [S-1][R][n][n], G = 16
    uint32_t *rcost = reinterpret_cast<uint32_t *>(smem + Ly.cost);   // [S-1][R * G][G], G < 16
    uint32_t *lmask = reinterpret_cast<uint32_t *>(smem + Ly.mask);   // [S-1][64], G = 16
    auto flow_of = [](uint32_t w) GWTF_INLINE { return (w >> W::flow) & W::mask; };
    auto cap_of = [](uint32_t w) GWTF_INLINE { return (w >> W::cap) & W::mask; };
    constexpr uint64_t kGroup = G == 16 ? 0xffffull : (1ull << G) - 1;

    // ---------------- ingest ----------------
    // `fits` turns false in some lane of a group for whatever the general form
    // has to see: values out of this form's bounds, invalid ones among them.
    const int64_t s0 = p.start_per_instance ? b : 0;
    const int supply = inst ? p.supply[b] : 0;
    bool fits = supply >= 0 && supply <= max_supply(false);
    uint32_t cin[MAXS][G], nw[MAXS], nc5[MAXS];
    uint32_t holes[MAXS]; // bit d: register d's link out of exit (k, j) is missing (G = 16: into node (k+1, j))
    uint32_t goal = uint32_t(max(supply, 0));
    uint32_t inflow[MAXS], outflow[MAXS];
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        nw[k] = nc5[k] = holes[k] = inflow[k] = outflow[k] = 0;
        if (k >= S) return;
        const int cp = node ? p.cap[size_t(b) * SN + k * n + j] : 0, w = node ? p.ncost[size_t(b) * SN + k * n + j] : 0;
        const int f = node ? p.nf0[size_t(s0) * SN + k * n + j] : 0;
        fits = fits && cp >= 0 && w >= 0 && w <= max_cost(false) && f >= 0 && f <= max_supply(false);
        goal = min(goal, group_sum<G>(uint32_t(min(max(cp, 0), 1 << 20))));
        nw[k] = uint32_t(f & 255) << W::flow | uint32_t(min(max(cp, 0), max_supply(false))) << W::cap;
        nc5[k] = uint32_t(min(max(w, 0), max_cost(false))) << 5;
    });
    each<MAXS - 1, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k + 1 >= S) return;
        uint32_t fl[G];
#pragma unroll
        for (int d = 0; d < G; ++d) {
            const int i = XOR ? j : d, jj = XOR ? j ^ d : j;
            const bool link = node && i < n && jj < n;
            const int a = link ? p.acost[(size_t(b) * (S - 1) + k) * nn + i * n + jj] : -1;
            const int f = link ? p.af0[(size_t(s0) * (S - 1) + k) * nn + i * n + jj] : 0;
            fits = fits && a >= -1 && a <= max_cost(false) && f >= 0 && f <= max_supply(false);
            holes[k] |= uint32_t(link && a < 0) << d;
            fl[d] = uint32_t(f & 255);
            const uint32_t c5 = uint32_t(min(max(a, 0), max_cost(false))) << 5;
            cin[k + 1][d] = a < 0 ? kNoLink : c5;
            if constexpr (XOR) {
                if (g < R) rcost[ridx(k, int(lane), d)] = c5 - kOff;
            } else {
                if (g < R && link) lcost[lidx(k, i, jj)] = uint16_t(c5);
            }
            if (g < R && link) lflow[lidx(k, i, jj)] = uint8_t(f);
        }
        // flow out of and into the nodes, for the check of conservation
        uint32_t row = 0, col = 0;
        if constexpr (XOR) {
#pragma unroll
            for (int d = 0; d < G; ++d) row += fl[d];
            turn<G>(fl);
#pragma unroll
            for (int d = 0; d < G; ++d) col += fl[d];
            turn<G>(cin[k + 1]);
        } else {
#pragma unroll
            for (int d = 0; d < G; ++d) {
                col += fl[d];
                const uint32_t sum = group_sum<G>(fl[d]);
                row = j == d ? sum : row;
            }
            lmask[k * 64 + lane] = 0;
        }
        outflow[k] = row;
        inflow[k + 1] = col;
    });
    const int srcc = node && p.src ? p.src[size_t(b) * n + j] : 0, snkc = node && p.snk ? p.snk[size_t(b) * n + j] : 0;
    const int sf = node ? p.sf0[size_t(s0) * n + j] : 0, tf = node ? p.tf0[size_t(s0) * n + j] : 0;
    fits = fits && srcc >= 0 && snkc >= 0 && srcc <= max_cost(false) && snkc <= max_cost(false);
    inflow[0] = uint32_t(sf);
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k >= S) return;
        if (k == S - 1) outflow[k] = uint32_t(tf);
        fits = fits && inflow[k] == flow_of(nw[k]) && outflow[k] == flow_of(nw[k]);
    });
    // a start flow of more than 255 units takes 32 bits nowhere but here
    uint32_t F = group_sum<G>(flow_of(nw[0]));
    fits = fits && F <= uint32_t(max_supply(false));
    const bool mine = inst && ((__ballot(!fits) >> gb) & kGroup) == 0;
    const uint32_t src5 = uint32_t(min(max(srcc, 0), max_cost(false))) << 5, snk5 = uint32_t(min(max(snkc, 0), max_cost(false))) << 5;
    bool give_up = false;   // the general form takes this instance after all
    // The walk table's flows are the node flows while stripping.
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k < S) table[k * 64 + lane] = nw[k];
    });
    __syncthreads();

    // ---------------- 1. strip ----------------
    int removed = 0;
    for (bool more = mine; __any(more);) {
        GWTF_PHASE;
        // The next node above its capacity, missing link with flow, or unit
        // above the supply, in that order, the lowest first.
        int k0 = -1, i0 = 0, k1 = 0, i1 = 0;
        uint32_t want = 0;
        for (int k = 0; k < S; ++k) {
            const uint32_t w = table[k * 64 + lane];
            const uint32_t over = more && flow_of(w) > cap_of(w) ? flow_of(w) - cap_of(w) : 0u;
            const uint32_t hit = uint32_t((__ballot(over > 0) >> gb) & kGroup);
            if (k0 < 0 && hit) {
                k0 = k1 = k;
                i0 = i1 = __builtin_ctz(hit);
                want = uint32_t(__shfl(int(over), gb + i0));
            }
        }
        each<MAXS - 1, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k + 1 >= S || !__any(more && k0 < 0 && holes[k] != 0)) return;
            // lowest missing link with flow among this lane's, as tail * 16 + head
            uint32_t low = ~0u;
            for (uint32_t m = more && k0 < 0 ? holes[k] : 0u; m; m &= m - 1) {
                const int d = __builtin_ctz(m), i = XOR ? j : d, jj = XOR ? j ^ d : j;
                if (lflow[lidx(k, i, jj)] > 0) low = min(low, uint32_t(i * 16 + jj));
            }
            low = group_min<G>(low);
            if (k0 < 0 && low != ~0u) {
                k0 = k;
                k1 = k + 1;
                i0 = int(low >> 4);
                i1 = int(low & 15u);
                want = uint32_t(lflow[lidx(k, i0, i1)]);
            }
        });
        if (k0 < 0 && F > uint32_t(max(supply, 0))) {
            const uint32_t hit = uint32_t((__ballot(more && flow_of(table[lane]) > 0) >> gb) & kGroup);
            k0 = k1 = 0;
            i0 = i1 = __builtin_ctz(hit | 1u << 31);
            want = F - uint32_t(supply);
        }
        more = more && k0 >= 0;
        if (!__any(more)) break;
        // Extend to both ends over the lowest link with flow; the path's node
        // of each stage goes to path[].
        const int at = (g < R ? g : 0) * kPathChunk;
        bool lost = false;
        if (more) {
            path[at + k0] = uint8_t(i0);
            path[at + k1] = uint8_t(i1);
        }
        int end = i0;
        for (int k = S - 1; k > 0; --k) {
            const bool step = more && k <= k0 && !lost;
            const uint32_t f = step && j < n ? uint32_t(lflow[lidx(k - 1, j, end)]) : 0u;
            const uint32_t hit = uint32_t((__ballot(f > 0) >> gb) & kGroup);
            if (step) {
                lost = hit == 0;
                end = lost ? end : __builtin_ctz(hit);
                path[at + k - 1] = uint8_t(end);
            }
        }
        end = i1;
        for (int k = 0; k + 1 < S; ++k) {
            const bool step = more && k >= k1 && !lost;
            const uint32_t f = step && j < n ? uint32_t(lflow[lidx(k, end, j)]) : 0u;
            const uint32_t hit = uint32_t((__ballot(f > 0) >> gb) & kGroup);
            if (step) {
                lost = hit == 0;
                end = lost ? end : __builtin_ctz(hit);
                path[at + k + 1] = uint8_t(end);
            }
        }
        wave_sync();
        uint32_t room = want;
        for (int k = j; k < S; k += G)
            if (more && !lost) {
                const int i = path[at + k];
                room = min(room, flow_of(table[k * 64 + gb + i]));
                if (k + 1 < S) room = min(room, uint32_t(lflow[lidx(k, i, path[at + k + 1])]));
            }
        const uint32_t delta = group_min<G>(room);
        if (more && (lost || delta == 0)) {
            give_up = true;
            more = false;
        }
        for (int k = j; k < S; k += G)
            if (more) {
                const int i = path[at + k];
                table[k * 64 + gb + i] -= delta << W::flow;
                if (k + 1 < S) {
                    const int e = lidx(k, i, path[at + k + 1]);
                    lflow[e] = uint8_t(lflow[e] - delta);
                }
            }
        wave_sync();
        F -= more ? delta : 0u;
        removed += more;
    }
    // what the flow left behind: node words and the residual reverse links
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k >= S) return;
        nw[k] = table[k * 64 + lane];
        if (k + 1 >= S || !node) return;
        for (int jj = 0; jj < n; ++jj) {
            if (lflow[lidx(k, j, jj)] == 0) continue;
            if constexpr (XOR) rcost[ridx(k, int(lane), j ^ jj)] += kOff;
            else lmask[k * 64 + lane] |= 1u << jj;
        }
    });
    __syncthreads();

    // ---------------- 2. cancel, 3. augment ----------------
    enum : int { kIdle = 0, kCancel = 1, kAugment = 2 };
    int mode = mine && !give_up ? kCancel : kIdle;
    int cycles = 0, augs = 0, rounds = 0;
    uint32_t din[MAXS], dout[MAXS], ncf[MAXS], ncr[MAXS];
    while (__any(mode != kIdle)) {
        uint32_t rc[XOR ? MAXS : 1][G];
        uint32_t ks = kKeyInf, kt = kKeyInf, srcr, snkr;
        {
            GWTF_PHASE;
            const uint32_t fresh = mode == kCancel ? (kZero | kRoot) : kKeyInf;
            ks = mode != kIdle ? (kZero | kRoot) : kKeyInf;
            kt = fresh;
            uint32_t last = 0;
            each<MAXS, false>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                din[k] = dout[k] = kKeyInf;
                if (k >= S) return;
                if (j < n) din[k] = dout[k] = fresh;
                const uint32_t fl = flow_of(nw[k]);
                ncf[k] = fl < cap_of(nw[k]) ? nc5[k] + kCodeSplit : kNoLink;
                ncr[k] = (fl > 0 ? nc5[k] : nc5[k] - kOff) - kCodeSplit;
                if (k == S - 1) last = fl;
                if constexpr (XOR) {
                    if (k + 1 < S) {
#pragma unroll
                        for (int d = 0; d < G; ++d) rc[k][d] = rcost[ridx(k, g < R ? int(lane) : j, d)];
                    }
                }
            });
            srcr = flow_of(nw[0]) > 0 ? src5 : src5 - kOff;
            snkr = (last > 0 ? snk5 : snk5 - kOff) - kCodeSrc;
        }
        bool found = false; // this group's cycle is listed
        int listed = 0;
        int search = 0;     // rounds of this search
        constexpr uint32_t kBegin = 1u << 31;
        uint32_t new_out = ~0u;  // stage k's exits (bit k), s (kBegin): changed since last read
        uint32_t new_in = ~0u;
        bool first = true;
        for (;;) {
            GWTF_PHASE;
            const uint32_t last = 1u << (S - 1);
            int lastk = -1; // stage of an exit of this lane that the backward sweep changed
            bool new_t = first;
            // -------- forward sweep --------
            new_out &= kBegin | (last - 1);
            if (!first) new_in = 0;
            each<MAXS, false>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                uint32_t best;
                if constexpr (k == 0) {
                    if (!(new_out & kBegin)) return;
                    best = label_of(ks) + src5 + kCodeSrc;
                } else {
                    if (!(new_out & (1u << (k - 1)))) return;
                    best = exchange<G, false, G>(label_of(dout[k - 1]) | uint32_t(j), cin[k]);
                }
                const bool better = j < n && best < label_of(din[k]);
                if (!__any(better)) return;
                din[k] = better ? best : din[k];
                new_in |= 1u << k;
                const uint32_t cand = label_of(din[k]) + ncf[k];
                const bool take = cand < label_of(dout[k]);
                dout[k] = take ? cand : dout[k];
                if (__any(take)) {
                    new_out |= (1u << k) & (last - 1);
                    if (k == S - 1) new_t = true;
                }
            });
            new_out = 0;
            // -------- t, then the backward sweep --------
            if (new_t) {
                uint32_t tk = kKeyInf;
                each<MAXS, false>([&](auto K) GWTF_INLINE {
                    constexpr int k = K;
                    if (k == S - 1) tk = dout[k];
                });
                tk = group_min<G>(j < n ? (label_of(tk) + snk5) | uint32_t(j) : kKeyInf);
                kt = tk < label_of(kt) ? tk : kt;
            }
            each<MAXS, true>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                if (k >= S) return;
                uint32_t best;
                if (k == S - 1) {
                    if (!new_t) return;
                    best = sub_tail(label_of(kt)) - snkr;
                } else {
                    if (!(new_in & (2u << k))) return;
                    constexpr int kn = k + 1 < MAXS ? k + 1 : k;
                    const uint32_t yr = sub_tail(label_of(din[kn])) | uint32_t(j);
                    if constexpr (XOR) {
                        best = exchange<G, true, G>(yr, rc[k]);
                    } else {
                        uint32_t rem = k + 1 < S ? lmask[k * 64 + lane] : 0u;
                        best = ~0u;
                        while (__any(rem != 0u)) {
                            const bool h0 = rem != 0u;
                            const int j0 = h0 ? __builtin_ctz(rem) : 0;
                            rem &= rem - 1u;
                            const bool h1 = rem != 0u;
                            const int j1 = h1 ? __builtin_ctz(rem) : 0;
                            rem &= rem - 1u;
                            const uint32_t y0 = uint32_t(__shfl(int(yr), gb + j0)), y1 = uint32_t(__shfl(int(yr), gb + j1));
                            const uint32_t c0 = h0 ? uint32_t(lcost[lidx(k, j, j0)]) : 0u;
                            const uint32_t c1 = h1 ? uint32_t(lcost[lidx(k, j, j1)]) : 0u;
                            best = h0 ? min(best, y0 - c0) : best;
                            best = h1 ? min(best, y1 - c1) : best;
                        }
                    }
                }
                const bool take = j < n && best < label_of(dout[k]);
                if (!__any(take) && !first) return;
                dout[k] = take ? best : dout[k];
                lastk = take ? k : lastk;
                if (__any(take)) new_out |= (1u << k) & (last - 1);
                const uint32_t cand = sub_tail(label_of(dout[k])) - ncr[k];
                const bool tin = j < n && cand < label_of(din[k]);
                din[k] = tin ? cand : din[k];
                if (__any(tin)) new_in |= 1u << k;
            });
            // s: only stage 0's entries lead back to it
            {
                const uint32_t sk = group_min<G>(j < n ? (sub_tail(label_of(din[0])) - srcr) | uint32_t(j) : kKeyInf);
                const bool less = sk < label_of(ks);
                ks = less ? sk : ks;
                if (__any(less)) new_out |= kBegin;
            }
            first = false;
            ++search;
            rounds += mode != kIdle && !found;
            if (new_out == 0) break;
            if (search >= kRoundCap) {
                give_up = give_up || (mode != kIdle && !found);
                mode = found ? mode : int(kIdle);
                break;
            }
            // -------- cycle check of the groups that still cancel --------
            if (search & 1) continue;
            const uint64_t hit = __ballot(lastk >= 0 && mode == kCancel && !found);
            if (hit == 0) continue;
            const uint32_t mine_hit = uint32_t((hit >> gb) & kGroup);
            const int v0 = mine_hit ? __builtin_ctz(mine_hit) : 0;
            const int sk0 = __shfl(lastk, gb + v0);
            const bool check = mine_hit != 0;
            if (check) {
                each<MAXS, false>([&](auto K) GWTF_INLINE {
                    constexpr int k = K;
                    if (k < S) table[k * 64 + lane] = ((dout[k] << 5) & 0x3e0u) | ((din[k] & 31u) | nw[k]);
                });
            }
            wave_sync();
            // one step back: from state (stage, node, at the exit) to the next
            // listed state; -1 at a root
            const int sroot = int(ks & 31u), troot = int(kt & 31u);
            auto back = [&](int st) GWTF_INLINE {
                const int k = (st >> 1) / G, v = (st >> 1) % G;
                const bool ex = (st & 1) != 0;
                const uint32_t w = table[k * 64 + gb + v];
                const uint32_t ce = (w >> 5) & 31u, ci = w & 31u;
                const bool via = ex && ce != kCodeSplit;
                const uint32_t code = via ? ce : ci;
                int nk = k, nv = int(code), nx = !via;
                if (code < 16) nk = via ? k + 1 : k - 1;
                else if (code == kCodeSplit) nv = v;       // reverse compute arc: the own exit
                else if (code == kCodeSrc) {               // by way of s or t
                    nk = via ? S - 1 : 0;
                    nv = via ? troot : sroot;
                    nx = via;
                    if (nv == int(kRoot)) return -1;
                } else return -1;
                return ((nk * G + nv) << 1) | nx;
            };
            int cyc = -1;
            if (check) {
                int turtle = ((sk0 * G + v0) << 1) | 1, hare = back(turtle), power = 1, len = 1;
                for (int steps = 0; hare >= 0 && hare != turtle && steps < 8 * (V + 2); ++steps) {
                    if (len == power) {
                        turtle = hare;
                        power *= 2;
                        len = 0;
                    }
                    hare = back(hare);
                    ++len;
                }
                cyc = hare == turtle ? hare : -1;
            }
            if (cyc >= 0) {
                int st = cyc;
                listed = 0;
                do {
                    path[g * kPathChunk + listed] = uint8_t(st);
                    ++listed;
                    st = back(st);
                } while (st != cyc && st >= 0 && listed < kPathChunk);
                found = true;
                if (st != cyc) { // longer than the list: the general form's
                    give_up = true;
                    mode = kIdle;
                    listed = 0;
                }
            }
            if (__any(cyc >= 0)) {
                each<MAXS, false>([&](auto K) GWTF_INLINE {
                    constexpr int k = K;
                    if (k >= S) return;
                    din[k] = cyc >= 0 ? kKeyInf : din[k];
                    dout[k] = cyc >= 0 ? kKeyInf : dout[k];
                });
                ks = cyc >= 0 ? kKeyInf : ks;
                kt = cyc >= 0 ? kKeyInf : kt;
            }
            wave_sync();
        }

        // -------- what each group pushes: its cycle, or its path --------
        GWTF_PHASE;
        const bool reach = mode == kAugment && kt < kFinite && F < goal;
        if (mode == kAugment && !reach) mode = kIdle;     // maximum flow
        const bool settled = mode == kCancel && !found;   // no negative cycle is left
        if (!found) {
            each<MAXS, false>([&](auto K) GWTF_INLINE {
                constexpr int k = K;
                if (k < S) table[k * 64 + lane] = ((dout[k] << 5) & 0x3e0u) | ((din[k] & 31u) | nw[k]);
            });
        }
        wave_sync();
        bool lost = false;
        if (reach) {
            int k = S - 1, v = int(kt & 31u);
            bool ex = true, go = true;
            listed = 0;
            while (go) {
                path[g * kPathChunk + listed] = uint8_t(((k * G + v) << 1) | int(ex));
                ++listed;
                const uint32_t w = table[k * 64 + gb + v];
                const uint32_t ce = (w >> 5) & 31u, ci = w & 31u;
                const bool via = ex && ce != kCodeSplit;
                const uint32_t code = via ? ce : ci;
                go = code <= kCodeSplit;
                lost = !go && (via || code != kCodeSrc);
                k += code == kCodeSplit ? 0 : (via ? 1 : -1);
                v = code == kCodeSplit ? v : int(code & 15u);
                ex = !via;
                if (go && (uint32_t(k) >= uint32_t(S) || listed == kPathChunk)) {
                    lost = true;
                    go = false;
                }
            }
        }
        const bool push = (reach && !lost) || (found && mode == kCancel);
        if (!push) listed = 0;
        wave_sync();
        auto each_listed = [&](auto f) GWTF_INLINE {
            for (int at = j; __any(at < listed); at += G) {
                if (at < listed) {
                    const int rec = int(path[g * kPathChunk + at]), k = (rec >> 1) / G, v = (rec >> 1) % G;
                    const int q = k * 64 + gb + v;
                    const uint32_t w = table[q];
                    const uint32_t ce = (w >> 5) & 31u, ci = w & 31u;
                    const bool ex = (rec & 1) != 0, via = ex && ce != kCodeSplit;
                    const bool link = (via ? ce : ci) < 16;
                    const int lk = via ? k : k - 1, tail = via ? v : int(ci), head = via ? int(ce) : v;
                    f(q, w, via, ex && !via, !via && ci == kCodeSplit, link, lk, tail, head);
                }
            }
        };
        uint32_t room = reach ? goal - F : kUnbounded;
        each_listed([&](int, uint32_t w, bool via, bool split, bool rev, bool link, int lk, int tail,
                        int head) GWTF_INLINE {
            if (split) room = min(room, cap_of(w) - flow_of(w));
            if (rev) room = min(room, flow_of(w));
            if (via && link) room = min(room, uint32_t(lflow[lidx(lk, tail, head)]));
        });
        const uint32_t delta = group_min<G>(room);
        if (lost || (push && (delta == 0 || delta == kUnbounded))) {
            give_up = true;
            mode = kIdle;
            listed = 0;
        }
        const bool apply = push && mode != kIdle;
        each_listed([&](int q, uint32_t, bool via, bool split, bool rev, bool link, int lk, int tail,
                        int head) GWTF_INLINE {
            if (split) atomicAdd(&table[q], delta << W::flow);
            if (rev) atomicSub(&table[q], delta << W::flow);
            if (link) {
                const int e = lidx(lk, tail, head);
                const uint32_t had = uint32_t(lflow[e]);
                lflow[e] = uint8_t(via ? had - delta : had + delta);
                if (had == (via ? delta : 0u)) { // the link empties or begins to carry flow
                    if constexpr (XOR) {
                        atomicAdd(&rcost[ridx(lk, gb + tail, tail ^ head)], via ? 0u - kOff : kOff);
                    } else {
                        uint32_t *mask = &lmask[lk * 64 + gb + tail];
                        if (via) atomicAnd(mask, ~(1u << head));
                        else atomicOr(mask, 1u << head);
                    }
                }
            }
        });
        wave_sync();
        each<MAXS, false>([&](auto K) GWTF_INLINE {
            constexpr int k = K;
            if (k < S) nw[k] = table[k * 64 + lane] & ~1023u;
        });
        if (apply) {
            cycles += mode == kCancel;
            augs += mode == kAugment;
            F += mode == kAugment ? delta : 0u;
        }
        if (mode == kCancel && rounds >= kTotalRounds) {
            give_up = true;
            mode = kIdle;
        }
        if (settled && mode == kCancel) mode = kAugment;
        if (mode == kAugment && F >= goal) mode = kIdle;
        wave_sync();
    }

    // ---------------- export ----------------
    if (!inst) return;
    if (!mine || give_up) {
        if (j == 0) p.status_out[b] = kChurnPassedOn;
        return;
    }
    const size_t na = size_t(S > 1 ? S - 1 : 0) * nn;
    uint32_t part = 0; // at most 2047 * 255 per arc and 2 + 8 * 17 arcs a lane, 16 lanes: below 2^32 for the group
    each<MAXS, false>([&](auto K) GWTF_INLINE {
        constexpr int k = K;
        if (k >= S) return;
        const uint32_t fl = flow_of(nw[k]);
        part += (nc5[k] >> 5) * fl;
        if (k == 0) part += (src5 >> 5) * fl;
        if (k == S - 1) part += (snk5 >> 5) * fl;
        if (j < n && p.nf_out) {
            p.nf_out[size_t(b) * SN + k * n + j] = int(fl);
            if (k == 0) p.sf_out[size_t(b) * n + j] = int(fl);
            if (k == S - 1) p.tf_out[size_t(b) * n + j] = int(fl);
        }
        if (k + 1 >= S) return;
        for (int e = j; e < nn; e += G) {
            const uint32_t f = lflow[lidx(k, 0, 0) + e];
            if (p.nf_out) p.af_out[size_t(b) * na + size_t(k) * nn + e] = int(f);
            if (f) {
                const int i = e / n, jj = e - i * n;
                if constexpr (XOR) part += (rcost[ridx(k, gb + i, i ^ jj)] >> 5) * f;
                else part += (uint32_t(lcost[lidx(k, i, jj)]) >> 5) * f;
            }
        }
    });
    part = group_sum<G>(part);
    if (j == 0) {
        p.F_out[b] = F;
        p.cost_out[b] = part;
        p.status_out[b] = GWTF_INST_OK;
        if (p.work) {
            p.work[4 * size_t(b) + 0] = removed;
            p.work[4 * size_t(b) + 1] = cycles;
            p.work[4 * size_t(b) + 2] = augs;
            p.work[4 * size_t(b) + 3] = rounds;
        }
    }
}

template <int G> hipError_t launch(const ChurnParams &p, const LaunchInfo &l, hipStream_t stream)
{
    const int R = rows_per_wave(64 / G, p.B, l.cus);
    const size_t lds = small_layout<kChurnPackedStages, G, false>(p.S, p.n, R).total;
    hipLaunchKernelGGL((churn_packed_kernel<G>), dim3(unsigned((p.B + R - 1) / R)), dim3(64), lds, stream, p, R);
    return hipGetLastError();
}

} // namespace

hipError_t launch_churn_packed(const ChurnParams &p, const LaunchInfo &l, hipStream_t stream)
{
    if (p.n <= 4) return launch<4>(p, l, stream);
    return p.n <= 8 ? launch<8>(p, l, stream) : launch<16>(p, l, stream);
}

} // namespace gwtf
