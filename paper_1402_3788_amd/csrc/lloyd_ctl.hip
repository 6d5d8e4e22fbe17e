// The iteration control block: reset at the start of a library call, and its
// report to the host.
#include "lloyd.h"

namespace lloyd {

namespace {

__global__ void ctl_reset_kernel(Ctl *ctl)
{
    int32_t *p = reinterpret_cast<int32_t *>(ctl);
    const int i = threadIdx.x;
    if (i < (int)(sizeof(Ctl) / sizeof(int32_t))) p[i] = 0;
}

// After iteration t (its centres launch has finished): records convergence the
// way the next iteration's first launch would, and copies the block to host
// memory. A copy of 256 bytes through the runtime costs the host several times
// a launch.
__global__ void ctl_report_kernel(Ctl *ctl, Ctl *host, int t, int fixed)
{
    const int i = threadIdx.x;
    if (!fixed && t >= 2 && ctl->converged_at == 0 && ctl->changed[t & 1] == 0) {
        __syncthreads();                       // (uniform: one workgroup, the same values)
        if (i == 0) ctl->converged_at = t;
        __syncthreads();
    }
    const int32_t v = reinterpret_cast<const int32_t *>(ctl)[i];
    __hip_atomic_store(reinterpret_cast<int32_t *>(host) + i, v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

hipError_t launch_ctl_report(Ctl *ctl, Ctl *host, int t, int fixed, hipStream_t s)
{
    hipLaunchKernelGGL(ctl_report_kernel, dim3(1), dim3(sizeof(Ctl) / sizeof(int32_t)), 0, s, ctl,
                       host, t, fixed);
    return hipGetLastError();
}

hipError_t launch_ctl_reset(Ctl *ctl, hipStream_t s)
{
    hipLaunchKernelGGL(ctl_reset_kernel, dim3(1), dim3(64), 0, s, ctl);
    return hipGetLastError();
}

}  // namespace lloyd
