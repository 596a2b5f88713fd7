// tiny_c64.hip - instantiations of the one-launch step (tiny_impl.h) for float2
// amplitudes.
#include "tiny_impl.h"

hipError_t tiny_c64(const GateArg &g, const PassBufs &b, hipStream_t s)
{
    if (g.m == 1) hipLaunchKernelGGL((sts_tiny::k_tiny<float2, 1>), dim3(1), dim3(sts_tiny::NT), 0, s, g, b);
    else if (g.m == 2) hipLaunchKernelGGL((sts_tiny::k_tiny<float2, 2>), dim3(1), dim3(sts_tiny::NT), 0, s, g, b);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

const void *tiny_c64_kernel(int m)
{
    return m == 1 ? reinterpret_cast<const void *>(&sts_tiny::k_tiny<float2, 1>)
                  : reinterpret_cast<const void *>(&sts_tiny::k_tiny<float2, 2>);
}
