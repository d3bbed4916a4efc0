// The packed pass for at most 4 nodes per stage, 4 lanes per instance
// (mcf_small_kernel.h).
#include "mcf_small_kernel.h"

namespace gwtf {

hipError_t launch_small_pass4(const SolveParams &p, size_t lds_max, hipStream_t s)
{
    return launch_group<4, 4>(p, lds_max, s);
}

} // namespace gwtf
