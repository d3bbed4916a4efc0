// The packed pass for at most 8 nodes per stage, 8 lanes per instance
// (mcf_small_kernel.h).
#include "mcf_small_kernel.h"

namespace gwtf {

hipError_t launch_small_pass8(const SolveParams &p, const LaunchInfo &l, hipStream_t s)
{
    return launch_group<8, 8>(p, l, s);
}

} // namespace gwtf
