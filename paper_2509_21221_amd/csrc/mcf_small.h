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
// lanes per instance, then 16 with a relaxation over that many rows.  With all
// 16 rows 11,880 instances of 12 x 9 took 3.88 ms and 40,320 of 8 x 13 4.95 ms,
// with 10 and 13 rows 3.63 and 4.87 ms.  They finish every instance of the batch.
hipError_t launch_small_pass4(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass8(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass10(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass13(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass16(const SolveParams &p, size_t lds_max, hipStream_t s);
inline hipError_t launch_small_pass(const SolveParams &p, size_t lds_max, hipStream_t s)
{
    if (p.n <= 4) return launch_small_pass4(p, lds_max, s);
    if (p.n <= 8) return launch_small_pass8(p, lds_max, s);
    if (p.n <= 10) return launch_small_pass10(p, lds_max, s);
    return p.n <= 13 ? launch_small_pass13(p, lds_max, s) : launch_small_pass16(p, lds_max, s);
}

} // namespace gwtf
