// Device pieces of the kernels that hold several instances per wave (the
// packed pass, mcf_small_kernel.h, and the packed churn re-solve,
// mcf_churn_packed.hip): keys, exchanges between the lanes of a group, the LDS
// layout.  mcf_small_kernel.h explains the mapping.
#pragma once

#include "mcf_device.h"

#include <utility>

namespace gwtf {
namespace {

using namespace dev;

constexpr uint32_t kFinite = 0x40000000u;     // labels (key & ~31) at or above are unreached
constexpr uint32_t kKeyInf = kFinite | 31u;   // an unreached vertex
constexpr uint32_t kNoLink = 0x40000000u;     // cost << 5 of a missing link
constexpr uint32_t kOff = 0x50000000u;        // taken off the cost of a reverse arc without flow
constexpr uint32_t kCodeSplit = 16, kCodeSrc = 17;
constexpr int kPathChunk = 64; // nodes of a path listed at a time
constexpr int64_t kSmallLabelLimit = (int64_t(1) << 25) - (int64_t(1) << 16);

// Largest cost and supply of each form.  A wide cost stays below 2^23 when
// labels stay below 2^25 (V >= 5), so cost << 5 is below 2^28.
constexpr int max_cost(bool wide) { return wide ? (1 << 23) - 1 : 2047; }
constexpr int max_supply(bool wide) { return wide ? 65535 : 255; }

// f(0), f(1), ... f(N - 1) (or the other way round) with the index a constant,
// so that arrays over the stages stay in registers.
#define GWTF_INLINE __attribute__((always_inline))
template <int N, bool DOWN, class Fn, int... I>
__device__ __forceinline__ void each_of(Fn &f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, DOWN ? N - 1 - I : I>{}), ...);
}
template <int N, bool DOWN, class Fn> __device__ __forceinline__ void each(Fn f)
{
    each_of<N, DOWN>(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ uint32_t label_of(uint32_t key) { return key & ~31u; }
// the label a cost is subtracted from: unreached moves to 2^31
__device__ __forceinline__ uint32_t sub_tail(uint32_t label) { return label + (label & kFinite); }

template <int CTRL> __device__ __forceinline__ uint32_t dpp(uint32_t x)
{
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), CTRL, 0xf, 0xf, true));
}
constexpr int kQuad1 = 0xb1, kQuad2 = 0x4e, kQuad3 = 0x1b, kHalfMirror = 0x141, kMirror = 0x140;

// Lane j ^ D of lane j's group of 4 or 8; m = the half-row mirror of x.
template <int D> __device__ __forceinline__ uint32_t xor_lane(uint32_t x, uint32_t m)
{
    if constexpr (D == 0) return x;
    else if constexpr (D == 1) return dpp<kQuad1>(x);
    else if constexpr (D == 2) return dpp<kQuad2>(x);
    else if constexpr (D == 3) return dpp<kQuad3>(x);
    else if constexpr (D == 4) return dpp<kQuad3>(m);
    else if constexpr (D == 5) return dpp<kQuad2>(m);
    else if constexpr (D == 6) return dpp<kQuad1>(m);
    else return m;
}

// c[d] of lane j becomes c[d] of lane j ^ d: rows of the links out of the
// nodes into columns of the links into them.
template <int G> __device__ __forceinline__ void turn(uint32_t (&c)[G])
{
#define GWTF_TURN(D)                                                                                                   \
    if constexpr (D < G) c[D % G] = xor_lane<D>(c[D % G], dpp<kHalfMirror>(c[D % G]))
    GWTF_TURN(1);
    GWTF_TURN(2);
    GWTF_TURN(3);
    GWTF_TURN(4);
    GWTF_TURN(5);
    GWTF_TURN(6);
    GWTF_TURN(7);
#undef GWTF_TURN
}

// min over the G lanes i of a group of (key of lane i) +- (cost of the link
// between lane i and this lane)
template <int G, bool SUB, int ROWS> __device__ __forceinline__ uint32_t exchange(uint32_t x, const uint32_t (&c)[ROWS])
{
    static_assert(((G == 4 || G == 8) && ROWS == G) || (G == 16 && ROWS <= 16 && !SUB), "group size");
    uint32_t v[ROWS];
    if constexpr (G == 16) {
#define GWTF_ROW(I)                                                                                                    \
    if constexpr (I < ROWS) v[I % ROWS] = dpp<0x150 + I>(x) + c[I % ROWS]
        GWTF_ROW(0); GWTF_ROW(1); GWTF_ROW(2); GWTF_ROW(3); GWTF_ROW(4); GWTF_ROW(5); GWTF_ROW(6); GWTF_ROW(7);
        GWTF_ROW(8); GWTF_ROW(9); GWTF_ROW(10); GWTF_ROW(11); GWTF_ROW(12); GWTF_ROW(13); GWTF_ROW(14); GWTF_ROW(15);
#undef GWTF_ROW
    } else {
        const uint32_t m = G == 8 ? dpp<kHalfMirror>(x) : 0u;
        auto arc = [](uint32_t k, uint32_t w) { return SUB ? k - w : k + w; };
        v[0] = arc(x, c[0]);
        v[1] = arc(xor_lane<1>(x, m), c[1]);
        v[2] = arc(xor_lane<2>(x, m), c[2]);
        v[3] = arc(xor_lane<3>(x, m), c[3]);
        if constexpr (G == 8) {
            v[4] = arc(xor_lane<4>(x, m), c[4]);
            v[5] = arc(xor_lane<5>(x, m), c[5]);
            v[6] = arc(xor_lane<6>(x, m), c[6]);
            v[7] = arc(m, c[7]);
        }
    }
    uint32_t best = v[0];
#pragma unroll
    for (int i = 1; i + 1 < ROWS; i += 2) best = min(min(best, v[i]), v[i + 1]);
    return ROWS % 2 == 0 ? min(best, v[ROWS - 1]) : best;
}

// min / max / sum over the G lanes of a group, in every lane of the group
template <int G, class Op> __device__ __forceinline__ uint32_t group_reduce(uint32_t v, Op op)
{
    v = op(v, dpp<kQuad1>(v));
    v = op(v, dpp<kQuad2>(v));
    if constexpr (G >= 8) v = op(v, dpp<kHalfMirror>(v));
    if constexpr (G == 16) v = op(v, dpp<kMirror>(v));
    return v;
}
template <int G> __device__ __forceinline__ uint32_t group_min(uint32_t v)
{
    return group_reduce<G>(v, [](uint32_t a, uint32_t b) { return min(a, b); });
}
template <int G> __device__ __forceinline__ int group_max(int v)
{
    return int(group_reduce<G>(uint32_t(v), [](uint32_t a, uint32_t b) { return uint32_t(max(int(a), int(b))); }));
}
template <int G> __device__ __forceinline__ uint32_t group_sum(uint32_t v)
{
    return group_reduce<G>(v, [](uint32_t a, uint32_t b) { return a + b; });
}

// Walk table word of a node: entry code, exit code << 5, then its flow and
// capacity (8 bits each, 16 when WIDE); for G < 16 also, in the top four bits of
// the low half, the number of links with flow out of it.
constexpr int kLinksAt = 28;
template <bool WIDE> struct Word {
    using type = uint32_t;
    static constexpr int flow = 10, cap = 18;
    static constexpr uint32_t mask = 0xff;
};
template <> struct Word<true> {
    using type = uint64_t;
    static constexpr int flow = 10, cap = 32;
    static constexpr uint32_t mask = 0xffff;
};
// Listed path node: (stage * G + node) << 1 | (the path comes to its exit).
template <bool BYTE> struct PathType { using type = uint8_t; };
template <> struct PathType<false> { using type = uint16_t; };

// LDS of one wave that holds R instances: the walk table [S][64], the listed
// path nodes [R][kPathChunk], the link flows [S-1][R][n][n], and the link
// costs: for G = 4 and 8 per exit the G words cost << 5 (less kOff without
// flow) of its links to nodes j ^ d, for G = 16 the costs << 5
// [S-1][R][n][n] and per exit the mask of its links with flow.  At eight 8 x 8
// instances a wave takes 20 KB, an eighth of a CU's LDS.
struct SmallLayout {
    size_t path, flow, cost, mask, total;
};
template <int MAXS, int G, bool WIDE> __host__ __device__ inline SmallLayout small_layout(int S, int n, int R)
{
    SmallLayout L;
    const size_t links = size_t(S > 1 ? S - 1 : 0) * R * n * n, pairs = size_t(S > 1 ? S - 1 : 0);
    size_t o = sizeof(typename Word<WIDE>::type) * S * 64;
    L.path = o;
    o += align16(sizeof(typename PathType<MAXS * G <= 128>::type) * R * kPathChunk);
    L.flow = o;
    o += align16((WIDE ? 2 : 1) * links);
    L.cost = o;
    if (G == 16) o += align16((WIDE ? 4 : 2) * links);
    else o += 4 * pairs * R * G * G;
    L.mask = o;
    if (G == 16) o += align16(4 * pairs * 64);
    L.total = o;
    return L;
}

__device__ __forceinline__ int opaque_s(int x)
{
    __asm__ volatile("" : "+s"(x));
    return x;
}
__device__ __forceinline__ unsigned opaque_v(unsigned x)
{
    __asm__ volatile("" : "+v"(x));
    return x;
}

    // The shape and the lane index as values the compiler cannot see through,
    // taken anew in each phase: what follows from them (addresses, stage
    // tests) is then computed where it is used instead of held in registers
    // across the whole solve, which would spill.  For kernels with parameters p
// and R instances per wave.
#define GWTF_PHASE                                                                                                     \
    const int S = opaque_s(p.S), n = opaque_s(p.n), nn = n * n;                                                        \
    const unsigned lane = opaque_v(threadIdx.x);                                                                       \
    const int g = int(lane / G), j = int(lane % G), gb = g * G /* first lane of the group */;                          \
    auto lidx = [=](int k, int i, int jj) GWTF_INLINE { return ((k * R + g) * n + i) * n + jj; };                      \
    auto ridx = [=](int k, int ln, int d) GWTF_INLINE { return (k * R * G + ln) * G + d; };                            \
    (void)S, (void)nn, (void)gb, (void)j, (void)lidx, (void)ridx

// Instances per wave of a batch: as few as keep it within one wave per SIMD of
// the device (four per CU), so that a small batch spreads over the device, and
// all groups of the wave beyond that.  On 256 CUs: 4,096 instances of 8 x 5
// (in the rest launch): 394 us within 512 waves, 375 within 1,024, 619 within
// 2,048; 1,024 of 4 x 4: 60, 59 and 59 us.
inline int rows_per_wave(int groups, int B, int cus)
{
    const int waves = 4 * (cus > 0 ? cus : 256);
    int R = 1;
    while (R < groups && (B + R - 1) / R > waves) R *= 2;
    return R;
}

} // namespace
} // namespace gwtf
