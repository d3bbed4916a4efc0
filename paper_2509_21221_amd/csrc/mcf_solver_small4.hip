// The packed pass for at most 4 nodes per stage, 4 lanes per instance
// (mcf_small_kernel.h).
#include "mcf_small_kernel.h"

namespace gwtf {

hipError_t launch_small_pass4(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    return launch_group<4, 4>(p, l, s);
}

} // namespace gwtf
