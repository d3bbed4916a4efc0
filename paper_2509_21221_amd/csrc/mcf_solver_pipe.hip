// Stage-pipelined register pass: one workgroup per instance, for pipelines of
// at most 32 stages of at most 64 nodes whose link costs fit in 16 bits.
//
// Same method as the other passes (successive shortest paths with Johnson
// potentials on the node-split stage graph, paper Sec. V-A Eq. 2), with the
// label-correcting step spread over the waves by stage instead of by row:
//
//  * Wave w owns P consecutive stages (k = w*P ...).  For each it keeps, in
//    vector registers, the 16-bit costs of every link into that stage (lane
//    j = receiving node, two rows per register: 32 registers per stage) and
//    the nodes' labels and predecessors (lane = node); capacities, compute
//    costs, node flows and the flow lists of the exits sit in LDS.
//  * Iteration t of stage k relaxes the links from stage k-1's exit labels
//    of the same iteration (only the rows whose label dropped since the stage
//    last saw them), applies its compute arcs in both directions and pulls
//    its reverse links from stage k+1's entry labels of iteration t-1.  A
//    wave sweeps its own stages in order, so a label crosses them within one
//    iteration; between waves the boundary stages' labels travel through LDS
//    mailboxes whose words carry the iteration's parity, and the reader waits
//    on the words themselves.  All waves run concurrently on different
//    stages, without workgroup barriers.
//  * Convergence travels with the labels: each exit-mailbox word of
//    iteration t also carries whether any stage up to that wave's last one
//    changed a label in iteration t, so the wave that owns the last stage
//    learns it for the whole pipeline and, when nothing changed, publishes
//    the sink's key and a stop word; the other waves leave on that word
//    while they wait for a mailbox.
//  * After convergence: potentials (kept in the device workspace), then wave
//    0 reads every node's predecessors, staged in LDS, into registers (one per
//    stage), walks the path over them and lists its nodes; its lanes take the
//    bottleneck, one node each, from the LDS node flows and flow lists, and
//    every wave applies the path to its own stages.
//
// What bounds it: the chain of stage steps, whose instructions a wave issues
// alone for most of a search (the first iteration passes through the waves one
// after another), with vector issue at 0.35 of the peak.  The keyed
// variant's step (predecessor in the key, residual compute arcs and the first
// four list entries in registers, two rows per instruction) and the walk over
// registers took 256 instances of 32 x 64 from 26.0 to 20.4 ms: label
// iterations 18.3 to 14.4, augmentations 2.65 to 1.98 ms per instance.
//
// Each mailbox is written by one wave and read by one other.  The reader of an
// exit mailbox (a wave's last-stage labels for iteration t) cannot be
// overtaken: the writer's iteration t+1 needs the reader's first-stage output
// of iteration t, which the reader publishes after its read, so a mailbox
// holds the awaited iteration or the one before it and one parity bit tells
// them apart.  The same holds for the entry mailboxes one iteration behind.
#include "mcf_device.h"
#include "mcf_pipe.h"

namespace gwtf {
namespace {

using namespace dev;

constexpr int kSpinLimit = 1 << 22;
constexpr uint32_t kNoArc16 = 0xffff;
constexpr int kBias = 1 << 30;
// Keyed variant.  A vertex is kept as key = label << 6 | row, where row is the
// exit (or, for an exit, the entry of the next stage) its label came over a
// link from; that it came over the node's compute arc is a bit of a wave-wide
// mask in scalar registers.  Finite keys stay below 2^30 (labels below 2^24).
// Unreached labels are 2^30, and 2^31 where a cost is subtracted from them; an
// arc without residual costs 2^30 forwards, and kOff less than its cost
// backwards: nothing that involves either lands in the finite range.
//
// With link costs of at most kPairMaxCost a relaxation takes two rows per
// instruction: 16-bit keys (label - base) << 6 | row, base a lower bound of the
// previous stage's exit labels, in saturating adds.  base is kept so close to
// the smallest of them that the row with that label gives every node a
// candidate of at most base + kPairMaxCost, so a sum that saturates is no
// improvement.  Larger costs take one row per
// instruction, a multiply-add of the cost's half register by 64.
constexpr uint32_t kKeyFinite = 0x40000000u;
constexpr uint32_t kKeyInf = kKeyFinite | 63u;
constexpr uint32_t kOff = 0x50000000u;
constexpr int kPairMaxCost = 1022;
constexpr int kListRegs = 4; // entries of an exit's flow list kept in registers during a search
__host__ __device__ constexpr bool keyed_fits(int64_t V, int64_t maxc) { return (V + 2) * maxc < (int64_t(1) << 24); }
__device__ __forceinline__ uint32_t key_base(uint32_t key) { return key & ~63u; }
__device__ __forceinline__ uint32_t sub_tail(uint32_t label) { return label + (label & kKeyFinite); }

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pair_add(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pair_min(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// 64 * (low or high half of w) + k
__device__ __forceinline__ uint32_t mad_lo64(uint32_t w, uint32_t k)
{
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, 64, %2" : "=v"(r) : "v"(w), "s"(k));
    return r;
}
__device__ __forceinline__ uint32_t mad_hi64(uint32_t w, uint32_t k)
{
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, 64, %2 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "s"(k));
    return r;
}

typedef uint32_t u32x32 __attribute__((ext_vector_type(32)));

__device__ __forceinline__ int key_label(uint64_t key) { return int(uint32_t(key >> 32)) - kBias; }

// The sink key of the wave: the smallest label and, among equal labels, the
// lowest lane; ~0 when no lane has one.
__device__ __forceinline__ uint64_t wave_min_key(bool has, int label)
{
    const uint32_t v = has ? uint32_t(label + kBias) : ~0u;
    const uint32_t m = wave_reduce_u32<false>(v);
    if (m == ~0u) return ~0ull;
    const int first = __builtin_ctzll(__ballot(v == m));
    return (uint64_t(m) << 32) | uint32_t(first);
}

// LDS accesses another wave may be racing with.
template <typename T> __device__ __forceinline__ T lds_ld(const T *p)
{
    return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T> __device__ __forceinline__ void lds_st(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Walk table word of a node: where its exit's and its entry's label came from
// (7 bits each: a row or partner below 64, or one of the codes).
constexpr uint32_t kFromSplit = 64, kFromSrc = 65, kFromNone = 127;
__device__ __forceinline__ uint32_t walk_word(uint32_t exit_from, uint32_t entry_from) { return exit_from | entry_from << 8; }
__device__ __forceinline__ uint32_t exit_from(uint32_t w) { return w & 127u; }
__device__ __forceinline__ uint32_t entry_from(uint32_t w) { return (w >> 8) & 127u; }
// A node whose exit is reached by its compute arc and its entry over a link.
__device__ __forceinline__ bool straight(uint32_t w) { return (w & (127u | kFromSplit << 8)) == kFromSplit; }
// Listed path node: its walk word, the node, the stage, and whether the path
// comes to its exit (then over to its entry if that is by the compute arc) or
// to its entry only.
__device__ __forceinline__ uint32_t path_node(uint32_t w, int k, int v, bool at_exit)
{
    return w | uint32_t(v) << 16 | uint32_t(k) << 22 | (at_exit ? 1u << 27 : 0u);
}
// Position of partner j in a flow list of `len` entries at `lo`, or -1; four
// entries per round of reads (a list has room past its last entry).
__device__ __forceinline__ int find_partner(const uint32_t *lent, int lo, int len, int j)
{
    int at = -1;
    for (int x = 0; x < len; x += 4) {
        uint32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = lent[lo + x + u];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (x + u < len && int(e[u] & 255u) == j) at = lo + x + u;
    }
    return at;
}

struct PathNode {
    int k, i, q;             // stage, node, k * 64 + i
    bool split, back;        // the path takes its compute arc, or that arc's reverse
    bool link_in, link_back; // it is entered over a link, or left over a reverse link
    int tail, head;          // link_in: tail exit of stage k-1; link_back: head entry of stage k+1
};
__device__ __forceinline__ PathNode path_unpack(uint32_t r)
{
    PathNode a;
    a.k = int((r >> 22) & 31u);
    a.i = int((r >> 16) & 63u);
    a.q = a.k * 64 + a.i;
    const bool at_exit = (r >> 27) & 1u;
    a.link_back = at_exit && exit_from(r) != kFromSplit;
    a.split = at_exit && !a.link_back;
    a.back = !a.link_back && entry_from(r) == kFromSplit;
    a.link_in = !a.link_back && entry_from(r) < kFromSplit;
    a.tail = int(entry_from(r) & 63u);
    a.head = int(exit_from(r) & 63u);
    return a;
}

// predecessors of one node, entry side in the low half, exit side in the high
__device__ __forceinline__ int pred_in(int pp) { return int(int16_t(pp & 0xffff)); }
__device__ __forceinline__ int pred_out(int pp) { return pp >> 16; }
__device__ __forceinline__ int pred_pack(int pi, int po) { return (pi & 0xffff) | (po << 16); }

struct PipeShared {
    unsigned long long final_key;
    int stop;  // iteration at which the search converged; 0 while it runs
    int fault; // a wait ran out, an iteration bound was exceeded, or a self-check failed
    int bad, wide, maxc;
    int plen, delta;
    int stage_tot[kPipeMaxStages];
    long long rows, pulls, steps;
    // kept by thread 0, here rather than in every wave's scalar registers
    long long cost, augs, rounds;
    uint64_t tick, clk_iter, clk_aug, clk_other;
    __device__ void lap(uint64_t &clock)
    {
        const uint64_t now = wall_clock64();
        clock += now - tick;
        tick = now;
    }
};

// Waits until all 64 words of a mailbox carry parity `par` in bit 0; returns
// this lane's word.  Sets why to 1 if the search stopped meanwhile, 2 if the
// wait ran out.  A wave that has its input raises its issue priority: the
// work between a mailbox read and the next mailbox write is what the other
// waves wait for, so it goes ahead of the three other waves on its SIMD
// (which are polling or doing work nobody waits for yet); the wave drops back
// at the start of its next iteration.
__device__ __forceinline__ uint32_t mailbox_wait(const uint32_t *mb, uint32_t par, const int *stop, int &why)
{
    const int lane = threadIdx.x & 63;
    for (int spins = 0;; ++spins) {
        const uint32_t v = lds_ld(&mb[lane]);
        if (__all((v & 1u) == par)) {
            __builtin_amdgcn_s_setprio(3);
            return v;
        }
        if (lds_ld(stop) != 0) {
            why = 1;
            return ~0u;
        }
        if (spins > kSpinLimit) {
            why = 2;
            return ~0u;
        }
        __builtin_amdgcn_s_sleep(4);
    }
}

template <int W, int P, bool kKeyed>
__global__ __launch_bounds__(64 * W, 1) void solve_pipe_kernel(SolveParams p)
{
    constexpr int NT = 64 * W;
    const int b = blockIdx.x;
    // the unscaled variant runs after the keyed one, on the instances it passed on
    if (!kKeyed && p.route[b] != kRoutePipeWide) return;
    const int S = p.S, n = p.n, SN = S * n, V = 2 * SN + 3;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = w * P;                 // this wave's first stage
    const int klast = min(S, k0 + P) - 1; // and last (k0 > klast for idle waves)
    const bool jv = lane < n;

    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ PipeShared ps;
    const PipeLayout L = pipe_layout(S, W, p.list_slots);
    uint32_t *exmb = reinterpret_cast<uint32_t *>(smem + L.exmb); // [W][64] last-stage exit labels << 2 | changed << 1 | parity
    uint32_t *enmb = reinterpret_cast<uint32_t *>(smem + L.enmb); // [W][64] first-stage entry labels << 1 | parity
    int *nf = reinterpret_cast<int *>(smem + L.nf);               // [S][64] node flow
    int *capl = reinterpret_cast<int *>(smem + L.capl);           // [S][64] node capacity
    int *ncl = reinterpret_cast<int *>(smem + L.ncl);             // [S][64] node compute cost
    uint32_t *words = reinterpret_cast<uint32_t *>(smem + L.words); // [S][64] walk table
    uint16_t *loff = reinterpret_cast<uint16_t *>(smem + L.loff); // [S][64]
    uint8_t *llen = reinterpret_cast<uint8_t *>(smem + L.llen);   // [S][64]
    uint32_t *path = reinterpret_cast<uint32_t *>(smem + L.path); // [2*S*64 + 40]
    int *lamt = reinterpret_cast<int *>(smem + L.lamt);           // flow of each list entry
    uint32_t *lent = reinterpret_cast<uint32_t *>(smem + L.lent); // partner | cost << 8

    const int32_t *gcap = p.cap + size_t(b) * SN;
    const int32_t *gnc = p.ncost + size_t(b) * SN;
    const int32_t *gac = S > 1 ? p.acost + size_t(b) * (S - 1) * n * n : nullptr;
    int32_t *gpot = p.pot + size_t(b) * V;
    const int supply = p.supply[b];

    if (tid == 0) {
        ps.bad = supply < 0;
        ps.wide = 0;
        ps.maxc = 0;
        ps.fault = 0;
        ps.rows = ps.pulls = ps.steps = 0;
        ps.cost = ps.augs = ps.rounds = 0;
        ps.clk_iter = ps.clk_aug = ps.clk_other = 0;
    }
    __syncthreads();

    // ---------------- ingest + validate ----------------
    u32x32 lw[P];
    int din[P], dout[P], pp[P];
    uint32_t holes = 0; // bit s: some link into stage k0+s is missing
    int srcc = 0, snkc = 0;
    {
        int bad = 0, wide = 0, mx = 0;
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const int k = k0 + s;
            const bool own = k <= klast;
            const int cp = (own && jv) ? gcap[k * n + lane] : 0;
            const int nc = (own && jv) ? gnc[k * n + lane] : 0;
            bad |= (cp < 0) | (nc < 0);
            mx = max(mx, nc);
            u32x32 v = (u32x32)(0xffffffffu);
            int hole = 0;
            if (own && k >= 1) {
                const int32_t *layer = gac + size_t(k - 1) * n * n;
#pragma unroll
                for (int r = 0; r < 32; ++r) {
                    const int a0 = (jv && 2 * r < n) ? layer[(2 * r) * n + lane] : -1;
                    const int a1 = (jv && 2 * r + 1 < n) ? layer[(2 * r + 1) * n + lane] : -1;
                    bad |= (a0 < -1) | (a1 < -1);
                    wide |= (a0 > 65534) | (a1 > 65534);
                    hole |= (jv & (2 * r < n) & (a0 < 0)) | (jv & (2 * r + 1 < n) & (a1 < 0));
                    mx = max(mx, max(a0, a1));
                    const uint32_t c0 = a0 < 0 ? kNoArc16 : uint32_t(min(a0, 65535));
                    const uint32_t c1 = a1 < 0 ? kNoArc16 : uint32_t(min(a1, 65535));
                    v[r] = c0 | (c1 << 16);
                }
            }
            lw[s] = v;
            if (__any(hole)) holes |= 1u << s;
            if (own) {
                capl[k * 64 + lane] = cp;
                ncl[k * 64 + lane] = nc;
                nf[k * 64 + lane] = 0;
                if (jv) {
                    gpot[3 + 2 * (k * n + lane)] = 0;
                    gpot[4 + 2 * (k * n + lane)] = 0;
                }
            }
        }
        if (k0 == 0 && jv && p.src) srcc = p.src[size_t(b) * n + lane];
        if (klast == S - 1 && k0 <= klast && jv && p.snk) snkc = p.snk[size_t(b) * n + lane];
        bad |= (srcc < 0) | (snkc < 0);
        mx = max(mx, max(srcc, snkc));
        if (__any(bad)) atomicOr(&ps.bad, 1);
        if (__any(wide)) atomicOr(&ps.wide, 1);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
        if (lane == 0) atomicMax(&ps.maxc, mx);
    }
    holes = __builtin_amdgcn_readfirstlane(holes);

    // flow-list capacity of each exit: min(cap, n, supply); none in the last stage
    {
        int base_of[P];
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const int k = k0 + s;
            const bool own = k <= klast && k < S - 1;
            const int cp = own ? capl[k * 64 + lane] : 0;
            const int c = (own && jv && supply > 0 && cp > 0) ? min(min(cp, n), supply) : 0;
            int incl = c;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int up = __shfl_up(incl, off);
                incl += lane >= off ? up : 0;
            }
            base_of[s] = incl - c;
            if (k <= klast && lane == 63) ps.stage_tot[k] = incl;
        }
        __syncthreads();
        long long before = 0;
        for (int kk = 0; kk < k0 && kk < S; ++kk) before += ps.stage_tot[kk];
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const int k = k0 + s;
            if (k > klast) break;
            loff[k * 64 + lane] = uint16_t(min<long long>(before + base_of[s], 65535));
            llen[k * 64 + lane] = 0;
            before += ps.stage_tot[k];
        }
        if (klast == S - 1 && k0 <= klast && lane == 0 && before > p.list_slots) atomicOr(&ps.wide, 2);
    }
    if (tid == 0) {
        gpot[0] = 0;
        gpot[1] = 0;
        gpot[2] = 0;
    }
    __syncthreads();
    int status = 0;
    if (ps.bad) status = 1;
    else if (int64_t(V) * ps.maxc >= kLabelBound) status = 2;
    if (status == 0 && ps.wide) {
        // 16-bit link costs or LDS lists do not fit: the fallback pass
        // solves this instance.
        if (tid == 0) p.route[b] = kRouteFallback;
        return;
    }
    if (kKeyed && status == 0 && !keyed_fits(V, ps.maxc)) {
        // labels too long for the keys: the unscaled variant solves this instance
        if (tid == 0) p.route[b] = kRoutePipeWide;
        return;
    }

    // keyed: link costs times 64 when two rows fit an instruction
    const bool pairs = kKeyed && ps.maxc <= kPairMaxCost;
    if (pairs) {
#pragma unroll
        for (int s = 0; s < P; ++s)
#pragma unroll
            for (int r = 0; r < 32; ++r) {
                const uint32_t v = lw[s][r];
                lw[s][r] = (v & 0x03ff03ffu) << 6 | ((v & 0xffffu) == kNoArc16 ? 0xffffu : 0u) |
                           (v >> 16 == kNoArc16 ? 0xffff0000u : 0u);
            }
    }

    int F = 0, pit = 0;
    bool fault = false;
    if (tid == 0) ps.tick = wall_clock64();

    // keyed: a lower bound of the exit labels of stage k0 + s - 1, at most
    // `slack` below the smallest.  Distances do not fall from one search to the
    // next, so what holds at the end of a search mostly serves the next one too.
    uint32_t base[P];
#pragma unroll
    for (int s = 0; s < P; ++s) base[s] = 0x80000000u; // above every label: set at the first relaxation
    const uint32_t slack = pairs ? uint32_t(kPairMaxCost - ps.maxc) << 6 : 0u;

    if (status == 0) {
        while (F < supply) {
            // ---- labels of a fresh search; mailboxes hold iteration 0 ----
            // The flow lists change only between searches: each exit's list
            // and the wave's longest list per stage are read once here.
            int lst_lo[P], lst_len[P], lst_max[P];
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int q = (k0 + s) * 64 + lane;
                const bool own = k0 + s <= klast && k0 + s + 1 < S;
                lst_lo[s] = own ? int(loff[q]) : 0;
                lst_len[s] = own && jv ? int(llen[q]) : 0;
                // keyed: only whether it is 0 and, above kListRegs, its value
                lst_max[s] = __any(lst_len[s] > (kKeyed ? kListRegs : 0)) ? int(wave_reduce_u32<true>(uint32_t(lst_len[s])))
                                                                       : int(__any(lst_len[s] > 0));
            }
            int seen[P], seeny[P];                   // unscaled variant
            uint32_t ki[P], ko[P], kseen[P], kseeny[P]; // keyed: entry and exit keys, last inputs
            uint32_t ncf[P], ncr[P], la[P][kListRegs], lc[P][kListRegs];
            uint64_t isplit[P], osplit[P];
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int k = k0 + s;
                din[s] = (k == 0 && jv) ? srcc : kInf;
                dout[s] = kInf;
                pp[s] = pred_pack(k == 0 ? kPredSrc : kPredNone, kPredNone);
                seen[s] = kInf;
                seeny[s] = kInf;
            }
            if (k0 <= klast && !kKeyed) {
                if (k0 >= 1) lds_st(&enmb[w * 64 + lane], uint32_t(din[0]) << 1);
                if (klast + 1 < S) lds_st(&exmb[w * 64 + lane], uint32_t(kInf) << 2);
            }
            if constexpr (kKeyed) {
#pragma unroll
                for (int s = 0; s < P; ++s) {
                    const int k = k0 + s, q = k * 64 + lane;
                    const bool own = k <= klast;
                    const int fl = own ? nf[q] : 0, cp = own ? capl[q] : 0, nc = own ? ncl[q] : 0;
                    ki[s] = (k == 0 && jv) ? uint32_t(srcc) << 6 : kKeyInf;
                    ko[s] = kKeyInf;
                    kseen[s] = kKeyFinite;
                    kseeny[s] = sub_tail(kKeyFinite);
                    ncf[s] = fl < cp ? uint32_t(nc) << 6 : kKeyFinite;
                    ncr[s] = (uint32_t(nc) << 6) - (fl > 0 ? 0u : kOff);
                    isplit[s] = osplit[s] = 0;
                    // the first entries of each exit's list: lane address of
                    // the partner, cost (a list has room past its last entry)
                    uint32_t ent[kListRegs];
#pragma unroll
                    for (int e = 0; e < kListRegs; ++e) ent[e] = lent[lst_lo[s] + e];
#pragma unroll
                    for (int e = 0; e < kListRegs; ++e) {
                        la[s][e] = (ent[e] & 63u) << 2;
                        lc[s][e] = e < lst_len[s] ? (ent[e] >> 8) << 6 : 0u - kOff;
                    }
                }
                if (k0 <= klast) {
                    if (k0 >= 1) lds_st(&enmb[w * 64 + lane], sub_tail(key_base(ki[0])));
                    if (klast + 1 < S) lds_st(&exmb[w * 64 + lane], kKeyFinite);
                }
            }
            if (tid == 0) {
                ps.stop = 0;
                ps.final_key = ~0ull;
            }
            __syncthreads();
            if (tid == 0) ps.lap(ps.clk_other);

            // ---- (1) pipelined label-correcting iterations ----
            uint32_t rows = 0, steps = 0;
            int pulls = 0;
            if constexpr (kKeyed) {
                for (int t = 1; k0 <= klast; ++t) {
                    if (t > 4 * V + 8) {
                        if (lane == 0) atomicOr(&ps.fault, 1);
                        break;
                    }
                    const uint32_t par = uint32_t(t) & 1u;
                    __builtin_amdgcn_s_setprio(0);
                    int why = 0;
                    uint64_t chg = 0;  // lanes with a changed label
                    uint32_t upch = 0; // 2 if a stage before this wave's changed in iteration t
#pragma unroll
                    for (int s = 0; s < P; ++s) {
                        const int k = k0 + s;
                        if (k > klast) break;
                        // links from stage k-1's exit labels X, then the node's compute arc
                        auto relax = [&](const uint32_t X) {
                            const uint64_t mask = __ballot(X < kseen[s]);
                            kseen[s] = min(kseen[s], X);
                            rows += __popcll(mask);
                            if (mask == 0) return;
                            const uint32_t mlo = uint32_t(mask), mhi = uint32_t(mask >> 32);
                            uint32_t best = kKeyInf;
                            // A group with a dropped row is taken whole: a row
                            // that did not drop was relaxed with the same label
                            // before, so it cannot beat the current one.
                            if ((holes >> s) & 1u) {
                                // some links are missing (cost 0xffff): skip them
                                const uint32_t xk = X | uint32_t(lane);
                                for (uint64_t m = mask; m; m &= m - 1) {
                                    const int r = __builtin_ctzll(m);
                                    const uint32_t c = (lw[s][r >> 1] >> (16 * (r & 1))) & 0xffffu;
                                    const uint32_t cand = __builtin_amdgcn_readlane(xk, r) + (pairs ? c : c << 6);
                                    best = c != kNoArc16 ? min(best, cand) : best;
                                }
                            } else if (pairs) {
                                if (__ballot(X < base[s]) != 0 || __ballot(X - base[s] <= slack) == 0)
                                    base[s] = wave_reduce_u32<false>(X);
                                const uint32_t rel = min(X - base[s], 0xffc0u) | uint32_t(lane);
                                const uint32_t two = rel | dpp_mov<0xb1, 0xf>(rel) << 16; // rows 2r and 2r + 1 in lane 2r
                                uint32_t acc0 = ~0u, acc1 = ~0u;
#pragma unroll
                                for (int g = 0; g < 8; ++g) {
                                    if ((g < 4 ? mlo : mhi) & (0xffu << (8 * (g & 3)))) {
                                        uint32_t x[4];
#pragma unroll
                                        for (int u = 0; u < 4; ++u) x[u] = __builtin_amdgcn_readlane(two, 8 * g + 2 * u);
#pragma unroll
                                        for (int u = 0; u < 4; u += 2) {
                                            acc0 = pair_min(acc0, pair_add(x[u], lw[s][4 * g + u]));
                                            acc1 = pair_min(acc1, pair_add(x[u + 1], lw[s][4 * g + u + 1]));
                                        }
                                    }
                                }
                                const uint32_t acc = pair_min(acc0, acc1);
                                best = base[s] + min(acc & 0xffffu, acc >> 16);
                            } else {
                                const uint32_t xk = X | uint32_t(lane);
#pragma unroll
                                for (int g = 0; g < 8; ++g) {
                                    if ((g < 4 ? mlo : mhi) & (0xffu << (8 * (g & 3)))) {
                                        uint32_t x[8];
#pragma unroll
                                        for (int u = 0; u < 8; ++u) x[u] = __builtin_amdgcn_readlane(xk, 8 * g + u);
#pragma unroll
                                        for (int u = 0; u < 8; u += 2) {
                                            const uint32_t wd = lw[s][(8 * g + u) >> 1];
                                            best = min(min(best, mad_lo64(wd, x[u])), mad_hi64(wd, x[u + 1]));
                                        }
                                    }
                                }
                            }
                            const bool better = jv && best < key_base(ki[s]);
                            const uint64_t took = __ballot(better);
                            if (took == 0) return;
                            ki[s] = better ? best : ki[s];
                            isplit[s] &= ~took;
                            chg |= took;
                        };
                        auto split_fwd = [&]() {
                            const uint32_t cand = key_base(ki[s]) + ncf[s];
                            const bool better = cand < key_base(ko[s]);
                            const uint64_t took = __ballot(better);
                            ko[s] = better ? cand : ko[s];
                            osplit[s] |= took;
                            chg |= took;
                        };
                        // reverse links, only when some entry label Y of stage k+1
                        // (unreached as 2^31) dropped since this stage last pulled;
                        // then the reverse compute arcs, whose tails change only here
                        auto pull = [&](const uint32_t Y) {
                            const uint64_t drop = __ballot(Y < kseeny[s]);
                            kseeny[s] = min(kseeny[s], Y);
                            if (drop == 0 || lst_max[s] == 0) return;
                            const int yk = int(Y | uint32_t(lane));
                            uint32_t v[kListRegs];
#pragma unroll
                            for (int e = 0; e < kListRegs; ++e) v[e] = uint32_t(__builtin_amdgcn_ds_bpermute(int(la[s][e]), yk)) - lc[s][e];
                            uint32_t best = min(min(v[0], v[1]), min(v[2], v[3]));
                            for (int e = kListRegs; e < lst_max[s]; e += 2) {
                                // the rest of a long list, from LDS
                                const bool h0 = e < lst_len[s], h1 = e + 1 < lst_len[s];
                                const uint32_t e0 = lent[lst_lo[s] + (h0 ? e : 0)], e1 = lent[lst_lo[s] + (h1 ? e + 1 : 0)];
                                const uint32_t y0 = uint32_t(__builtin_amdgcn_ds_bpermute(int((e0 & 63u) << 2), yk));
                                const uint32_t y1 = uint32_t(__builtin_amdgcn_ds_bpermute(int((e1 & 63u) << 2), yk));
                                best = h0 ? min(best, y0 - (e0 >> 8 << 6)) : best;
                                best = h1 ? min(best, y1 - (e1 >> 8 << 6)) : best;
                            }
                            pulls += lst_len[s];
                            const bool better = best < key_base(ko[s]);
                            const uint64_t took = __ballot(better);
                            if (took == 0) return;
                            ko[s] = better ? best : ko[s];
                            osplit[s] &= ~took;
                            const uint32_t cand = sub_tail(key_base(ko[s])) - ncr[s];
                            const bool less = cand < key_base(ki[s]);
                            const uint64_t took2 = __ballot(less);
                            ki[s] = less ? cand : ki[s];
                            isplit[s] |= took2;
                            chg |= took | took2;
                        };
                        // The input held by this wave first (a wave's first stage
                        // pulls from its second's entry labels of iteration t-1,
                        // its second relaxes from its first's exit labels of
                        // iteration t), then the one another wave sends: the work
                        // between a mailbox read and the next mailbox write is
                        // what the waves pass to each other.
                        if (s < P - 1 && k + 1 < S) pull(sub_tail(key_base(ki[s + 1 < P ? s + 1 : s])));
                        if (s > 0) relax(key_base(ko[s > 0 ? s - 1 : 0]));
                        if (s == 0 && k >= 1) {
                            // exit labels of stage k-1, iteration t, from the previous wave
                            const uint32_t word = mailbox_wait(&exmb[(w - 1) * 64], par, &ps.stop, why);
                            if (why) break;
                            upch = __builtin_amdgcn_readfirstlane(word) & 2u;
                            relax(key_base(word));
                        }
                        split_fwd();
                        if (s == P - 1 && k + 1 < S) {
                            // entry labels of stage k+1, iteration t-1, from the next wave
                            const uint32_t Y = mailbox_wait(&enmb[(w + 1) * 64], par ^ 1u, &ps.stop, why) & ~63u;
                            if (why) break;
                            pull(Y);
                        }
                        ++steps;
                        if (s == 0 && k >= 1) lds_st(&enmb[w * 64 + lane], sub_tail(key_base(ki[s])) | par);
                        if (k == klast && k + 1 < S)
                            lds_st(&exmb[w * 64 + lane], key_base(ko[s]) | upch | (chg ? 2u : 0u) | par);
                    }
                    if (why) {
                        if (why == 2 && lane == 0) atomicOr(&ps.fault, 1);
                        break;
                    }
                    // the wave of the last stage: no label changed anywhere in
                    // iteration t ends the search
                    if (klast == S - 1 && upch == 0 && chg == 0) {
                        uint32_t last = kKeyInf;
#pragma unroll
                        for (int s = 0; s < P; ++s)
                            if (k0 + s == S - 1) last = ko[s];
                        const uint64_t skey = wave_min_key(jv && last < kKeyFinite, int(last >> 6) + snkc);
                        if (lane == 0) {
                            ps.final_key = skey;
                            lds_st(&ps.stop, t);
                        }
                        break;
                    }
                }
                // labels and predecessors as the phases below take them
#pragma unroll
                for (int s = 0; s < P; ++s) {
                    const bool ri = ki[s] < kKeyFinite, ro = ko[s] < kKeyFinite;
                    din[s] = ri ? int(ki[s] >> 6) : kInf;
                    dout[s] = ro ? int(ko[s] >> 6) : kInf;
                    const int pi = ((isplit[s] >> lane) & 1u) ? kPredSplit : (k0 + s == 0 ? kPredSrc : int(ki[s] & 63u));
                    const int po = ((osplit[s] >> lane) & 1u) ? kPredSplit : int(ko[s] & 63u);
                    pp[s] = pred_pack(ri ? pi : kPredNone, ro ? po : kPredNone);
                }
            }
            if (k0 <= klast && !kKeyed) {
                for (int t = 1;; ++t) {
                    if (t > 4 * V + 8) {
                        if (lane == 0) atomicOr(&ps.fault, 1);
                        break;
                    }
                    const uint32_t par = uint32_t(t) & 1u;
                    __builtin_amdgcn_s_setprio(0);
                    int why = 0;
                    bool chg = false;
                    uint32_t upch = 0; // 2 if a stage before this wave's changed in iteration t
                    uint64_t skey = ~0ull;
#pragma unroll
                    for (int s = 0; s < P; ++s) {
                        const int k = k0 + s;
                        if (k > klast) break;
                        const int q = k * 64 + lane;
                        const int fl = nf[q], cp = capl[q], nc = ncl[q];
                        int di = din[s], dq = dout[s], pi = pred_in(pp[s]), po = pred_out(pp[s]);
                        const int di0 = di, dq0 = dq;
                        // links from stage k-1's exit labels X
                        auto relax = [&](const int X) {
                            const bool dr = X < seen[s];
                            seen[s] = dr ? X : seen[s];
                            const uint64_t mask = __ballot(dr);
                            rows += __popcll(mask);
                            // rows that dropped, two per cost register, in row order
                            if (mask) {
                                if (!((holes >> s) & 1u)) {
                                    // one scalar test per group of 8 rows, then one
                                    // bit test per row of a group that has any
                                    const uint32_t mlo = uint32_t(mask), mhi = uint32_t(mask >> 32);
#pragma unroll
                                    for (int g = 0; g < 8; ++g) {
                                        const uint32_t half = g < 4 ? mlo : mhi;
                                        if (half & (0xffu << (8 * (g & 3)))) {
#pragma unroll
                                            for (int r = 8 * g; r < 8 * g + 8; ++r) {
                                                if (half & (1u << (r & 31))) {
                                                    const uint32_t wd = lw[s][r >> 1];
                                                    const int cand = __builtin_amdgcn_readlane(X, r) + int((r & 1) ? wd >> 16 : wd & 0xffffu);
                                                    pi = cand < di ? r : pi;
                                                    di = min(di, cand);
                                                }
                                            }
                                        }
                                    }
                                } else {
                                    // some links are missing (cost 0xffff): skip them
                                    uint64_t m = mask;
                                    while (m) {
                                        const int r = __builtin_ctzll(m);
                                        m &= m - 1;
                                        const uint32_t c = (lw[s][r >> 1] >> (16 * (r & 1))) & 0xffffu;
                                        const int cand = __builtin_amdgcn_readlane(X, r) + int(c);
                                        const bool take = (c != kNoArc16) & (cand < di);
                                        pi = take ? r : pi;
                                        di = take ? cand : di;
                                    }
                                }
                            }
                        };
                        // reverse links, only when some entry label of stage k+1 dropped
                        // since this stage last pulled (lists change only between
                        // searches): four list entries per pass, partner labels from
                        // the partner's lane (the loop runs to the wave's longest
                        // list so every cross-lane read has all lanes active)
                        auto pull = [&](const int Y) {
                            const bool ydr = Y < seeny[s];
                            seeny[s] = ydr ? Y : seeny[s];
                            if (k + 1 < S && __ballot(ydr) != 0) {
                                const int lo = lst_lo[s], len = lst_len[s], maxlen = lst_max[s];
                                for (int e = 0; e < maxlen; e += 4) {
                                    uint32_t ent[4];
#pragma unroll
                                    for (int u = 0; u < 4; ++u) ent[u] = lent[lo + e + u];
                                    // the four partner reads first, then the updates as
                                    // selects, so the reads are in flight together
                                    int dj[4];
#pragma unroll
                                    for (int u = 0; u < 4; ++u) dj[u] = __shfl(Y, e + u < len ? int(ent[u] & 255u) : 0);
#pragma unroll
                                    for (int u = 0; u < 4; ++u) {
                                        const int cand = dj[u] - int(ent[u] >> 8);
                                        const bool take = (e + u < len) & (dj[u] < kInf) & (cand < dq);
                                        dq = take ? cand : dq;
                                        po = take ? int(ent[u] & 255u) : po;
                                    }
                                }
                                pulls += len;
                            }
                        };
                        auto split_rev = [&]() {
                            if (fl > 0 && dq < kInf && dq - nc < di) {
                                di = dq - nc;
                                pi = kPredSplit;
                            }
                        };
                        auto split_fwd = [&]() {
                            if (di < kInf && fl < cp && di + nc < dq) {
                                dq = di + nc;
                                po = kPredSplit;
                            }
                        };
                        // The input held by this wave first (a wave's first stage
                        // pulls from its second's entry labels of iteration t-1,
                        // its second relaxes from its first's exit labels of
                        // iteration t), then the one another wave sends: the work
                        // between a mailbox read and the next mailbox write is
                        // what the waves pass to each other.
                        if (s < P - 1 && k + 1 < S) {
                            pull(din[s + 1]);
                            split_rev();
                        }
                        if (s > 0) relax(dout[s - 1]);
                        if (s == 0 && k >= 1) {
                            // exit labels of stage k-1, iteration t, from the previous wave
                            const uint32_t word = mailbox_wait(&exmb[(w - 1) * 64], par, &ps.stop, why);
                            if (why) break;
                            upch = __builtin_amdgcn_readfirstlane(word) & 2u;
                            relax(int(word >> 2));
                        }
                        split_rev();
                        split_fwd();
                        if (s == P - 1 && k + 1 < S) {
                            // entry labels of stage k+1, iteration t-1, from the next wave
                            const int Y = int(mailbox_wait(&enmb[(w + 1) * 64], par ^ 1u, &ps.stop, why) >> 1);
                            if (why) break;
                            pull(Y);
                            split_rev();
                        }
                        ++steps;
                        chg |= (di != di0) | (dq != dq0);
                        din[s] = di;
                        dout[s] = dq;
                        pp[s] = pred_pack(pi, po);
                        if (s == 0 && k >= 1) lds_st(&enmb[w * 64 + lane], (uint32_t(di) << 1) | par);
                        if (k == klast && k + 1 < S) {
                            const uint32_t ch = (upch | (__any(chg) ? 2u : 0u));
                            lds_st(&exmb[w * 64 + lane], (uint32_t(dq) << 2) | ch | par);
                        }
                        if (k == S - 1) {
                            skey = wave_min_key(jv && dq < kInf, dq + snkc);
                        }
                    }
                    if (why) {
                        if (why == 2 && lane == 0) atomicOr(&ps.fault, 1);
                        break;
                    }
                    // the wave of the last stage: no label changed anywhere in
                    // iteration t ends the search
                    if (klast == S - 1 && upch == 0 && !__any(chg)) {
                        if (lane == 0) {
                            ps.final_key = skey;
                            lds_st(&ps.stop, t);
                        }
                        break;
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) pulls += __shfl_xor(pulls, off);
            if (lane == 0) {
                atomicAdd(reinterpret_cast<unsigned long long *>(&ps.rows), (unsigned long long)rows);
                atomicAdd(reinterpret_cast<unsigned long long *>(&ps.steps), (unsigned long long)steps);
                atomicAdd(reinterpret_cast<unsigned long long *>(&ps.pulls), (unsigned long long)pulls);
            }
            __syncthreads();
            if (tid == 0) ps.lap(ps.clk_iter);
            if (ps.fault) {
                fault = true;
                break;
            }
            const uint64_t fk = ps.final_key;
            if (tid == 0) ps.rounds += ps.stop;
            if (fk == ~0ull) break; // sink unreachable: the flow is maximum

            // ---- (2) stage predecessors ----
            const int Dt = key_label(fk), predt = __builtin_amdgcn_readfirstlane(int(uint32_t(fk)));
            const int dred = Dt - pit;
            // The lane index, opaque here so that the per-lane addresses and
            // words below are computed after each search rather than held in
            // registers across the label iterations (which would spill them).
            int ln = lane;
            __asm__ volatile("" : "+v"(ln));
#pragma unroll
            for (int s = 0; s < P; ++s) {
                const int k = k0 + s;
                if (k > klast) break;
                const int pi = pred_in(pp[s]), po = pred_out(pp[s]);
                const uint32_t from_in = pi == kPredSplit ? kFromSplit : pi == kPredSrc ? kFromSrc : pi >= 0 ? uint32_t(pi) : kFromNone;
                const uint32_t from_out = po == kPredSplit ? kFromSplit : po >= 0 ? uint32_t(po) : kFromNone;
                words[k * 64 + ln] = walk_word(from_out, from_in);
            }
            __syncthreads();
            // potentials of this wave's nodes; wave 0 reads its own before its
            // walk and writes them after it
            auto update_potentials = [&]() {
#pragma unroll
                for (int s = 0; s < P; ++s) {
                    const int k = k0 + s;
                    if (k <= klast && jv) {
                        int32_t *pin = gpot + 3 + 2 * (k * n + ln);
                        pin[0] = min(din[s], pin[0] + dred);
                        pin[1] = min(dout[s], pin[1] + dred);
                    }
                }
            };
            if (w != 0) update_potentials();

            // ---- (3) wave 0 walks the predecessors, then the whole wave
            // takes the bottleneck over the listed nodes ----
            if (w == 0) {
                // Lane i holds the words of node i of every stage, so a run over
                // straight nodes takes a register and a lane read and a few
                // scalar instructions per node instead of a read of the table
                // in LDS and its way to a scalar register.
                u32x32 mine;
#pragma unroll
                for (int kk = 0; kk < W * P; ++kk) mine[kk] = words[min(kk, S - 1) * 64 + ln];
                int len = 0, k = S - 1, v = predt;
                bool at_exit = true, okw = predt >= 0 && predt < n;
                while (okw) {
                    if (at_exit) {
                        const int k1 = k, v1 = v;
                        uint32_t met = 0;
                        for (;;) {
                            k = __builtin_amdgcn_readfirstlane(k);
                            v = __builtin_amdgcn_readfirstlane(v);
                            const uint32_t wd = __builtin_amdgcn_readlane(mine[k], v);
                            if (!straight(wd)) break; // stage 0 has none: its entries come from the data node
                            met = ln == k ? wd : met;
                            v = int(entry_from(wd));
                            k -= 1;
                        }
                        // lanes k + 1 .. k1 hold the nodes met; each one's index
                        // is in the word of the node before it
                        const uint32_t before = __shfl_down(met, 1);
                        if (ln > k && ln <= k1)
                            path[len + k1 - ln] = path_node(met, ln, ln == k1 ? v1 : int(entry_from(before)), true);
                        len += k1 - k;
                    }
                    const uint32_t wd = __builtin_amdgcn_readfirstlane(words[k * 64 + v]);
                    path[len] = path_node(wd, k, v, at_exit);
                    ++len;
                    const uint32_t ce = exit_from(wd), ci = entry_from(wd);
                    if (at_exit && ce != kFromSplit) { // on by a reverse link
                        okw = ce < 64 && k + 1 < S;
                        k += 1;
                        v = int(ce);
                        at_exit = false;
                    } else if (ci == kFromSplit) { // by the reverse compute arc
                        at_exit = true;
                    } else {
                        if (ci == kFromSrc) break;
                        okw = ci < 64 && k >= 1;
                        k -= 1;
                        v = int(ci);
                        at_exit = true;
                    }
                    okw = okw && len <= 2 * SN + 4;
                }
                if (lane == 0) ps.plen = okw ? len : -1;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                int r = supply - F;
                for (int e = lane; e < len; e += 64) {
                    const PathNode a = path_unpack(path[e]);
                    if (a.split) r = min(r, capl[a.q] - nf[a.q]);
                    if (a.back) r = min(r, nf[a.q]);
                    if (a.link_back) {
                        const int at = find_partner(lent, loff[a.q], llen[a.q], a.head);
                        r = min(r, at >= 0 ? lamt[at] : 0);
                    }
                }
                r = int(wave_reduce_u32<false>(uint32_t(r)));
                if (lane == 0) ps.delta = r;
                update_potentials();
            }
            __syncthreads();
            const int len = ps.plen, delta = ps.delta;
            if (len < 0 || delta <= 0) {
                fault = true;
                break;
            }

            // ---- (4) each wave applies the path to its stages ----
            // (a link belongs to its tail's stage; links that empty come before
            // links that fill, so a list never holds more than its slots)
            if (k0 <= klast) {
                for (int pass = 0; pass < 2; ++pass) {
                    for (int e = lane; e < len; e += 64) {
                        const PathNode a = path_unpack(path[e]);
                        const bool own = a.k >= k0 && a.k <= klast;
                        if (pass == 0) {
                            if (!own) continue;
                            if (a.split) nf[a.q] += delta;
                            if (a.back) nf[a.q] -= delta;
                            if (a.link_back) {
                                const int lo = loff[a.q], hi = lo + llen[a.q];
                                const int le = find_partner(lent, lo, hi - lo, a.head);
                                if (le < 0 || lamt[le] < delta) {
                                    atomicOr(&ps.fault, 1);
                                } else if (lamt[le] == delta) { // the arc empties: move the last entry here
                                    lent[le] = lent[hi - 1];
                                    lamt[le] = lamt[hi - 1];
                                    llen[a.q] = uint8_t(hi - 1 - lo);
                                } else {
                                    lamt[le] -= delta;
                                }
                            }
                        } else if (a.link_in && a.k - 1 >= k0 && a.k - 1 <= klast) {
                            const int kt = a.k - 1, q = kt * 64 + a.tail;
                            const int lo = loff[q], hi = lo + llen[q];
                            const int le = find_partner(lent, lo, hi - lo, a.i);
                            if (le >= 0) {
                                lamt[le] += delta;
                            } else if (hi - lo >= min(min(capl[q], n), supply)) {
                                atomicOr(&ps.fault, 1);
                            } else {
                                lent[hi] = uint32_t(a.i) | (uint32_t(gac[(size_t(kt) * n + a.tail) * n + a.i]) << 8);
                                lamt[hi] = delta;
                                llen[q] = uint8_t(hi + 1 - lo);
                            }
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            F += delta;
            pit = Dt;
            // No barrier here: a wave's lists and node flows are its own, and
            // what the next search resets was last read two barriers ago.
            if (tid == 0) {
                ps.cost += (long long)delta * Dt;
                ps.augs++;
                ps.lap(ps.clk_aug);
            }
        }
        __syncthreads();
        fault = fault || ps.fault != 0;
    }

    // ---------------- export ----------------
    // The launch's parameters read again from here: pointers used only below
    // then take no scalar registers in the searches.
    __attribute__((address_space(4))) const SolveParams *again =
        (__attribute__((address_space(4))) const SolveParams *)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(again));
    const bool ok = status == 0 && !fault;
    int32_t *nfo = again->node_flow + size_t(b) * SN;
    if (k0 <= klast && jv) {
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const int k = k0 + s;
            if (k <= klast) {
                const int q = k * n + lane;
                nfo[q] = ok ? nf[k * 64 + lane] : 0;
                if (!ok) {
                    gpot[3 + 2 * q] = 0;
                    gpot[4 + 2 * q] = 0;
                }
            }
        }
    }
    const size_t na = size_t(S - 1) * n * n;
    int32_t *af = again->arc_flow + size_t(b) * na;
    for (size_t e = tid; e < na; e += NT) af[e] = 0;
    __syncthreads();
    if (ok) {
        for (int q = tid; q < (S - 1) * 64; q += NT) {
            const int k = q >> 6, i = q & 63;
            if (i >= n) continue;
            for (int e = loff[q]; e < loff[q] + llen[q]; ++e) af[(size_t(k) * n + i) * n + (lent[e] & 255u)] = lamt[e];
        }
    }
    if (tid == 0) {
        gpot[0] = 0;
        gpot[1] = 0;
        gpot[2] = ok ? pit : 0;
        again->F_out[b] = ok ? F : 0;
        again->cost_out[b] = ok ? ps.cost : 0;
        again->status_out[b] = status != 0 ? status : (fault ? kStatusInternal : 0);
        again->route[b] = kRouteReg;
        int64_t *st = again->stats + size_t(b) * kStatsPerInstance;
        const double ns_per_tick = 1e6 / double(again->clock_khz > 0 ? again->clock_khz : 100000);
        st[0] = ps.augs;
        st[1] = ps.rounds;
        st[2] = ps.rows;
        st[3] = ps.pulls;
        st[4] = int64_t(double(ps.clk_iter) * ns_per_tick);
        st[5] = 0;
        st[6] = int64_t(double(ps.clk_aug) * ns_per_tick);
        st[7] = int64_t(double(ps.clk_other) * ns_per_tick);
        st[8] = ps.steps;
        st[9] = 0;
    }
}

// Waves and stages per wave for a pipeline of S stages.
void pipe_shape(int S, int &W, int &P)
{
    if (S <= 8) {
        W = 8;
        P = 1;
    } else if (S <= 16) {
        W = 16;
        P = 1;
    } else {
        W = 16;
        P = 2;
    }
}

} // namespace

bool pipe_pass_fits(int S, int n) { return S >= 1 && S <= kPipeMaxStages && n >= 1 && n <= 64; }

int64_t pipe_pass_slots(int S, size_t lds_max)
{
    int W, P;
    pipe_shape(S, W, P);
    const size_t fixed = pipe_layout(S, W, 0).total + sizeof(PipeShared) + 256;
    if (fixed >= lds_max) return 0;
    return std::min<int64_t>(int64_t((lds_max - fixed) / 8), 65535);
}

hipError_t launch_pipe_pass(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    int W, P;
    pipe_shape(p.S, W, P);
    const size_t lds = pipe_layout(p.S, W, p.list_slots).total;
    // keyed variant first; the unscaled one takes the instances it passed on
    if (W == 8) {
        hipLaunchKernelGGL((solve_pipe_kernel<8, 1, true>), dim3(p.B), dim3(512), lds, s, p);
        if (!l.first_only)
            hipLaunchKernelGGL((solve_pipe_kernel<8, 1, false>), dim3(p.B), dim3(512), lds, s, p);
    } else if (P == 1) {
        hipLaunchKernelGGL((solve_pipe_kernel<16, 1, true>), dim3(p.B), dim3(1024), lds, s, p);
        if (!l.first_only)
            hipLaunchKernelGGL((solve_pipe_kernel<16, 1, false>), dim3(p.B), dim3(1024), lds, s, p);
    } else {
        hipLaunchKernelGGL((solve_pipe_kernel<16, 2, true>), dim3(p.B), dim3(1024), lds, s, p);
        if (!l.first_only)
            hipLaunchKernelGGL((solve_pipe_kernel<16, 2, false>), dim3(p.B), dim3(1024), lds, s, p);
    }
    return hipGetLastError();
}

} // namespace gwtf
