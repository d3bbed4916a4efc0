// The packed pass for at most 10 nodes per stage, 16 lanes per instance
// (mcf_small_kernel.h).
#include "mcf_small_kernel.h"

namespace gwtf {

hipError_t launch_small_pass10(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    return launch_group<16, 10>(p, l, s);
}

} // namespace gwtf
