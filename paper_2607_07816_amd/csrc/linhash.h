// linhash.h - the bucket hash of a bucketed state: a fixed linear map over
// GF(2) from 64-bit keys to 32 bits, of which the top hb bits are the bucket.
//
// Because the map is linear, a gate moves terms between buckets in a way that
// does not depend on the term: key bit q flips the hash by lin_dir(q), so the
// 2^m partners of a term lie in the 2^m buckets b ^ span(dirs of the gate's
// qubits), and so do its new terms. A state kept in bucket order therefore
// needs no sort before a gate: a workgroup reads one coset of buckets, and
// its survivors are the new contents of the same buckets.
//
// The directions are pseudo-random (SplitMix64 outputs); the seed is one for
// which every window of hb + 6 consecutive qubits, hb = 4..22, has full rank,
// so that a state filling all keys of such a window loads every bucket
// alike.
#pragma once

#include "common.h"

constexpr u32 lin_dir(int q)
{
    u64 x = 33ull * 64ull + (u64)q + 0x9e3779b97f4a7c15ull;
    x ^= x >> 30;
    x *= 0xbf58476d1ce4e5b9ull;
    x ^= x >> 27;
    x *= 0x94d049bb133111ebull;
    x ^= x >> 31;
    return (u32)(x >> 32);
}

// the key bits whose parity is bit `bit` (0..31) of the hash
constexpr u64 lin_mask(int bit)
{
    u64 m = 0;
    for (int q = 0; q < 64; ++q) m |= (u64)((lin_dir(q) >> bit) & 1u) << q;
    return m;
}

#define STS_LIN4(i) lin_mask(i), lin_mask((i) + 1), lin_mask((i) + 2), lin_mask((i) + 3)
static __constant__ const u64 k_lin_masks[32] = {STS_LIN4(0),  STS_LIN4(4),  STS_LIN4(8),  STS_LIN4(12),
                                                 STS_LIN4(16), STS_LIN4(20), STS_LIN4(24), STS_LIN4(28)};

__device__ __forceinline__ u32 sts_parity(u64 key, u64 mask)
{
    return (u32)(__popc((u32)key & (u32)mask) + __popc((u32)(key >> 32) & (u32)(mask >> 32))) & 1u;
}

// bits [from, from + NB) of the hash of key
template <int NB> __device__ __forceinline__ u32 lin_bits(u64 key, int from)
{
    u32 v = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) v |= sts_parity(key, k_lin_masks[from + i]) << i;
    return v;
}

// Bucket geometry of one gate on a state of 2^hb buckets. A workgroup's tile
// is a coset of the 4-dimensional span of E[0..3], a wave's share (four
// buckets) a coset of span(E[0], E[1]), which holds the gate's directions.
// The extra directions are the previous gate's, whose buckets lie next to
// each other in memory.
#define STS_BKT_DIMS 4
struct BktPlan {
    int hb;    // bucket bits of the input
    int delta; // further bits of the output (the state grew): hb + delta
    u32 E[STS_BKT_DIMS];   // basis; E[i] has bit p_i set, later ones are zero there
    int piv[STS_BKT_DIMS]; // the pivots p_i, ascending
    u64 cm[2];             // coordinate of a key along E[0], E[1]: parity(key & cm)
    u64 rm[4];             // refinement bits of the output bucket (bit i: parity(key & rm[i]))
};

// bucket of tile t with all coordinates zero
__device__ __forceinline__ u32 bkt_rep(const BktPlan &p, u32 t)
{
#pragma unroll
    for (int i = 0; i < STS_BKT_DIMS; ++i) {
        const u32 low = (1u << p.piv[i]) - 1u;
        t = ((t & ~low) << 1) | (t & low);
    }
    return t;
}

__device__ __forceinline__ u32 bkt_comb(const BktPlan &p, u32 c)
{
    u32 v = 0;
#pragma unroll
    for (int i = 0; i < STS_BKT_DIMS; ++i) v ^= (c >> i) & 1u ? p.E[i] : 0u;
    return v;
}

// Host side: the plan of a gate on qubits q[0..m-1] (m <= 2) for hb >= 4
// bucket bits, with the previous gate's qubits as the preferred extras.
inline BktPlan bkt_plan(int hb, int delta, int m, const int *q, int pm, const int *pq)
{
    BktPlan p{};
    p.hb = hb;
    p.delta = delta;
    u32 pv[STS_BKT_DIMS] = {};
    int n = 0;
    auto add = [&](u32 v) {
        if (n == STS_BKT_DIMS) return;
        for (int i = 0; i < n; ++i)
            if ((v >> pv[i]) & 1u) v ^= p.E[i];
        if (!v) return;
        int top = 31;
        while (!((v >> top) & 1u)) --top;
        p.E[n] = v;
        pv[n] = (u32)top;
        ++n;
    };
    for (int t = 0; t < m; ++t) add(lin_dir(q[t]) >> (32 - hb));
    // the wave's two dimensions are reduced against each other, so that their
    // coordinates are read off their pivots
    for (int t = 0; t < pm; ++t) add(lin_dir(pq[t]) >> (32 - hb));
    for (int i = 0; i < hb; ++i) add(1u << i);
    if ((p.E[0] >> pv[1]) & 1u) p.E[0] ^= p.E[1];
    // coordinates of each key bit
    for (int t = 0; t < 64; ++t) {
        const u32 r = lin_dir(t) >> (32 - hb);
        for (int i = 0; i < 2; ++i) p.cm[i] |= (u64)((r >> pv[i]) & 1u) << t;
    }
    for (int i = 0; i < delta && i < 4; ++i) p.rm[i] = lin_mask(32 - hb - delta + i);
    for (int i = 0; i < STS_BKT_DIMS; ++i) p.piv[i] = (int)pv[i];
    for (int i = 0; i < STS_BKT_DIMS; ++i)
        for (int j = i + 1; j < STS_BKT_DIMS; ++j)
            if (p.piv[j] < p.piv[i]) {
                const int t = p.piv[i];
                p.piv[i] = p.piv[j];
                p.piv[j] = t;
            }
    return p;
}
