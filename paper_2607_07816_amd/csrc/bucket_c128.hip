// bucket_c128.hip - instantiations of the bucketed gate step (bucket_impl.h) for
// double2 amplitudes; compiled as a unit of its own so the library builds in
// parallel.
#include <algorithm>

#include "bucket_impl.h"

hipError_t bucket_c128_pass(int kind, int m, const PassBufs &b, int tiles, hipStream_t s, const GateArg *first)
{
    switch (m) {
    case 1: return sts_bucket::launch_m<double2, 1>(kind, b, tiles, s, first);
    case 2: return sts_bucket::launch_m<double2, 2>(kind, b, tiles, s, first);
    }
    return hipErrorInvalidValue;
}

int bucket_c128_groups(int m, int tiles)
{
    using namespace sts_bucket;
    return m == 1 ? weigh_grid<double2, 1>(tiles) : weigh_grid<double2, 2>(tiles);
}

const void *bucket_c128_first(int kind, int m)
{
    return m == 1 ? sts_bucket::first_kernel<double2, 1>(kind) : sts_bucket::first_kernel<double2, 2>(kind);
}
