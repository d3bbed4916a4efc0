// Internal interface of the packed small-instance pass (mcf_solver_small.hip):
// one to sixteen instances per wave, for at most 16 stages of at most 16
// nodes.  Not part of the public C ABI.
#pragma once

#include "mcf_internal.h"

namespace gwtf {

constexpr int kPackedStages = 8;    // reported as the packed pass (and its rest as the fallback)
constexpr int kSmallMaxStages = 16; // deeper pipelines up to here are reported as the LDS pass
inline bool small_pass_fits(int S, int n) { return S >= 1 && S <= kSmallMaxStages && n <= 16; }
// Both launches of the pass with 4, 8 or 16 lanes per instance (n at most
// that); they finish every instance of the batch.
hipError_t launch_small_pass4(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass8(const SolveParams &p, size_t lds_max, hipStream_t s);
hipError_t launch_small_pass16(const SolveParams &p, size_t lds_max, hipStream_t s);
inline hipError_t launch_small_pass(const SolveParams &p, size_t lds_max, hipStream_t s)
{
    if (p.n <= 4) return launch_small_pass4(p, lds_max, s);
    return p.n <= 8 ? launch_small_pass8(p, lds_max, s) : launch_small_pass16(p, lds_max, s);
}

} // namespace gwtf
