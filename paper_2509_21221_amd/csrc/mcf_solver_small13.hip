// The packed pass for at most 13 nodes per stage, 16 lanes per instance
// (mcf_small_kernel.h).
#include "mcf_small_kernel.h"

namespace gwtf {

hipError_t launch_small_pass13(const SolveParams &p, size_t lds_max, hipStream_t s)
{
    return launch_group<16, 13>(p, lds_max, s);
}

} // namespace gwtf
