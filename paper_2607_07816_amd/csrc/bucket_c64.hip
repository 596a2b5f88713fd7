// bucket_c64.hip - instantiations of the bucketed gate step (bucket_impl.h) for
// float2 amplitudes; compiled as a unit of its own so the library builds in
// parallel.
#include <algorithm>

#include "bucket_impl.h"

hipError_t bucket_c64_pass(int kind, int m, const PassBufs &b, int tiles, hipStream_t s)
{
    switch (m) {
    case 1: return sts_bucket::launch_m<float2, 1>(kind, b, tiles, s);
    case 2: return sts_bucket::launch_m<float2, 2>(kind, b, tiles, s);
    }
    return hipErrorInvalidValue;
}

int bucket_c64_capacity(int m)
{
    return m == 1 ? sts_bucket::hist_capacity_b<float2, 1>() : sts_bucket::hist_capacity_b<float2, 2>();
}
