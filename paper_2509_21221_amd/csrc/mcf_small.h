// Internal interface of the packed small-instance pass (mcf_small_kernel.h):
// one to sixteen instances per wave, for at most 16 stages of at most 16
// nodes.  Not part of the public C ABI.
#pragma once

#include "mcf_internal.h"

namespace gwtf {

constexpr int kPackedStages = 8;    // reported as the packed pass (and its rest as the fallback)
constexpr int kSmallMaxStages = 16; // deeper pipelines up to here are reported as the LDS pass
inline bool small_pass_fits(int S, int n) { return S >= 1 && S <= kSmallMaxStages && n <= 16; }
// The launches of the pass, for n at most the number in the name: 4 and 8
// lanes per instance, then 16 with a relaxation over that many rows.  In turn
// with a build that always takes all 16: 4,096 instances of 12 x 9 1.24 against
// 1.30 ms, 16,384 of 8 x 10 1.60 / 1.65 (10 rows); 16,384 of 8 x 13 2.29 / 2.33,
// 4,096 of 12 x 13 2.10 / 2.16, 40,320 placements of 8 x 13 4.69 / 4.77 (13 rows),
// quartiles within 0.3 % of these.  They finish every instance of the batch.
hipError_t launch_small_pass4(const SolveParams &p, const LaunchInfo &l, hipStream_t s);
hipError_t launch_small_pass8(const SolveParams &p, const LaunchInfo &l, hipStream_t s);
hipError_t launch_small_pass10(const SolveParams &p, const LaunchInfo &l, hipStream_t s);
hipError_t launch_small_pass13(const SolveParams &p, const LaunchInfo &l, hipStream_t s);
hipError_t launch_small_pass16(const SolveParams &p, const LaunchInfo &l, hipStream_t s);
inline hipError_t launch_small_pass(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    if (p.n <= 4) return launch_small_pass4(p, l, s);
    if (p.n <= 8) return launch_small_pass8(p, l, s);
    if (p.n <= 10) return launch_small_pass10(p, l, s);
    return p.n <= 13 ? launch_small_pass13(p, l, s) : launch_small_pass16(p, l, s);
}

} // namespace gwtf
