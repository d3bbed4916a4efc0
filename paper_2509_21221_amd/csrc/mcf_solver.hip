// Batched min-cost max-flow on layered stage graphs: the kernels of the LDS
// and fallback passes (the method is in mcf_solve_body.h) and the export of
// the data node's flows.
#include "mcf_solve_body.h"

namespace gwtf {
namespace {

using namespace dev;

// One workgroup per instance, or per instance the passes before handed on
// (route_all tells): narrow state in LDS (n <= 64), or wide state in device
// memory.
template <int WAVES, bool NARROW>
__global__ __launch_bounds__(WAVES * 64) void solve_kernel(SolveParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.x;
    if (!p.route_all && p.route[b] != kRouteFallback) return;
    solve_body<WAVES, NARROW>(p, b, NARROW ? kRouteLds : kRouteGlobal, smem);
}

__global__ void export_kernel(const int32_t *nf, int32_t S, int32_t n, int32_t first, int32_t count,
                              int32_t *src_flow, int32_t *snk_flow)
{
    size_t idx = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= size_t(count) * n) return;
    size_t b = idx / n, j = idx % n;
    const int32_t *f = nf + (size_t(first) + b) * S * n;
    if (src_flow) src_flow[idx] = f[j];
    if (snk_flow) snk_flow[idx] = f[size_t(S - 1) * n + j];
}

constexpr int kFallbackWaves = 16;

} // namespace

int fallback_waves() { return kFallbackWaves; }

hipError_t set_lds_limits(size_t max_bytes)
{
    hipError_t e = hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(solve_kernel<1, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(max_bytes));
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(solve_kernel<4, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(max_bytes));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(solve_kernel<kFallbackWaves, false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(max_bytes));
}

hipError_t launch_lds_pass(const SolveParams &p, int waves, size_t lds_bytes, hipStream_t s)
{
    if (waves == 1)
        hipLaunchKernelGGL((solve_kernel<1, true>), dim3(p.B), dim3(64), lds_bytes, s, p);
    else
        hipLaunchKernelGGL((solve_kernel<4, true>), dim3(p.B), dim3(256), lds_bytes, s, p);
    return hipGetLastError();
}

hipError_t launch_fallback_pass(const SolveParams &p, size_t lds_bytes, hipStream_t s)
{
    hipLaunchKernelGGL((solve_kernel<kFallbackWaves, false>), dim3(p.B), dim3(kFallbackWaves * 64),
                       lds_bytes, s, p);
    return hipGetLastError();
}

hipError_t launch_export(const int32_t *node_flow_ws, int32_t S, int32_t n, int32_t first, int32_t count,
                         int32_t *src_flow, int32_t *snk_flow, hipStream_t s)
{
    size_t total = size_t(count) * n;
    if (total == 0) return hipSuccess;
    unsigned blocks = unsigned((total + 255) / 256);
    hipLaunchKernelGGL(export_kernel, dim3(blocks), dim3(256), 0, s, node_flow_ws, S, n, first, count,
                       src_flow, snk_flow);
    return hipGetLastError();
}

} // namespace gwtf
