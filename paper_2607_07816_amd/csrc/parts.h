// parts.h - the parts of a share that is larger than a wave's tables.
//
// Every part holds the terms whose mixed masked key (sts_mix64, 64 bits) has
// one prefix. The walk goes through the prefixes in order, depth first: from
// `base` bits, at which evenly spread terms fit, a part that does not fit is
// split into its two halves, and once both are done the walk is back at the
// shallower prefix. A cluster of terms with a long common prefix therefore
// costs two parts per bit of it and leaves the other parts as they are.
#pragma once

#include "common.h"

struct PartWalk {
    int base, depth; // bits of the shallowest prefix, and of this one
    u64 pre;         // this prefix

    // a share of n terms, in parts of at most cap
    __host__ __device__ __forceinline__ void begin(u32 n, u32 cap)
    {
        base = 0;
        pre = 0;
        if (n > cap)
            while ((n >> base) > cap * 3 / 4) ++base;
        depth = base;
    }
    // instead of this part, its first half (at 64 bits a part is one group)
    __host__ __device__ __forceinline__ void split()
    {
        ++depth;
        pre <<= 1;
    }
    // to the next part; false: this was the last
    __host__ __device__ __forceinline__ bool next()
    {
        while (depth > base && (pre & 1ull)) {
            pre >>= 1;
            --depth;
        }
        ++pre;
        return depth > base || pre < (1ull << base);
    }
};
