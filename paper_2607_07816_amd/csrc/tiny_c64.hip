// tiny_c64.hip - instantiations of the one-launch step (tiny_impl.h) for float2
// amplitudes.
#include "tiny_impl.h"

hipError_t tiny_c64(const GateArg &g, const PassBufs &b, u64 n_bound, hipStream_t s)
{
    switch (g.m) {
    case 1: return sts_tiny::launch<float2, 1>(g, b, n_bound, s);
    case 2: return sts_tiny::launch<float2, 2>(g, b, n_bound, s);
    }
    return hipErrorInvalidValue;
}

const void *tiny_c64_kernel(int m, int size)
{
    return m == 1 ? sts_tiny::kernel<float2, 1>(size) : sts_tiny::kernel<float2, 2>(size);
}
