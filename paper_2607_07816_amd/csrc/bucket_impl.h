// bucket_impl.h - the gate step of a bucketed state (gates of 1 and 2 qubits).
//
// The state is kept in 2^hb buckets by a hash that is linear over GF(2)
// (linhash.h), each bucket one contiguous run of terms. A gate's partners lie
// in the four buckets of one coset of span(E[0], E[1]), and so do its new
// terms, so the step needs no sort: each wave reads the four runs of its
// coset (about 256 terms), groups them in a hash table of its own in LDS, and
// multiplies the groups out; the survivors go back to the same four buckets.
// A wave works alone - no barriers in the tile loop - so that the waves of a
// CU hide each other's chains of LDS round trips.
//
// A share larger than the LDS tables (the hash is uneven there) is taken in
// several parts, each with the groups whose second hash has one prefix
// (parts.h); every part scans the whole share.
#pragma once
#include "group_impl.h"
#include "parts.h"
#include "select_impl.h"

namespace sts_bucket {

using namespace sts_group;

constexpr int BW = STS_WG / 64;    // waves of a workgroup, each with a share of its own
constexpr int BW_CAP = 320;        // terms of a share staged at once
constexpr int BW_SLOTS = 512;      // hash slots of a wave
constexpr int BW_ROUNDS = BW_CAP / 64;
constexpr u32 BW_BINNED = 640;     // larger shares bypass the LDS bins (their sums are bounded by this)
constexpr int BW_FLUSH = 16;       // tiles between flushes of the LDS bins

// a wave's tables
template <typename AT> struct WaveSmem {
    AT amp[BW_CAP];
    u64 key[BW_CAP];
    unsigned long long slot[BW_SLOTS]; // a group: the staged index + 1 of its member j at bit 16 j
    unsigned short lead[BW_CAP];       // from the front: the only member of each group of one; from the end: the
                                       // slots of the others
    unsigned short hard[64];
};

template <typename AT, int NW> struct BktSmem {
    WaveSmem<AT> w[NW];
    AT ucol[16]; // U by columns: U[i][j] at [2^m j + i]
};

// orders a wave's own LDS accesses (which the hardware performs in order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// (HIP's __ballot goes through an integer: two more instructions a call)
__device__ __forceinline__ u64 wballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ u32 uni(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }

// what the grouping needs of the gate, read once: through the argument block
// every use would be a load of its own, since the kernel's stores might
// change it
template <int M> struct GateLoc {
    u64 nm;           // key bits outside the gate
    u64 bit[M];       // the gate's key bits
    int q[M];
};

template <int M> __device__ __forceinline__ GateLoc<M> gate_loc(const GateArg &g)
{
    GateLoc<M> l;
    l.nm = ~0ull;
#pragma unroll
    for (int t = 0; t < M; ++t) {
        l.q[t] = (int)uni((u32)g.q[t]);
        l.bit[t] = 1ull << l.q[t];
        l.nm &= ~l.bit[t];
    }
    return l;
}

// a key's pattern on the gate's qubits, and a pattern's key bits
template <int M> __device__ __forceinline__ u32 pattern_of(const GateLoc<M> &l, u64 key)
{
    u32 j = 0;
#pragma unroll
    for (int t = 0; t < M; ++t) j |= (u32)((key >> l.q[t]) & 1ull) << t;
    return j;
}

template <int M> __device__ __forceinline__ u64 pattern_bits(const GateLoc<M> &l, int i)
{
    u64 k = 0;
#pragma unroll
    for (int t = 0; t < M; ++t) k |= ((i >> t) & 1) ? l.bit[t] : 0ull;
    return k;
}

// the four runs of a wave's share (in scalar registers)
struct Share {
    u32 o0, d1, d2, d3; // first term of run 0; what further runs add to it, less their starts in the flat index
    u32 p1, p2, p3, n;  // starts of runs 1..3 in the flat index; terms in all
};

// lane i % 4 reads the bounds of run i
__device__ __forceinline__ uint2 load_runs(const BktPlan &p, const uint2 *__restrict__ bd, u32 tile, int wv)
{
    return bd[bkt_rep(p, tile) ^ bkt_comb(p, ((u32)sts_lane() & 3u) | ((u32)wv << 2))];
}

// the share whose runs four lanes hold, from lane `at` on
__device__ __forceinline__ Share share_of(uint2 d, int at = 0)
{
    u32 beg[4], cnt[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        beg[i] = (u32)__builtin_amdgcn_readlane((int)d.x, at + i);
        cnt[i] = (u32)__builtin_amdgcn_readlane((int)d.y, at + i) - beg[i];
    }
    Share s;
    s.p1 = cnt[0];
    s.p2 = s.p1 + cnt[1];
    s.p3 = s.p2 + cnt[2];
    s.n = s.p3 + cnt[3];
    s.o0 = beg[0];
    s.d1 = beg[1] - s.p1 - beg[0];
    s.d2 = beg[2] - s.p2 - (beg[1] - s.p1);
    s.d3 = beg[3] - s.p3 - (beg[2] - s.p2);
    return s;
}

__device__ __forceinline__ Share load_share(const BktPlan &p, const uint2 *__restrict__ bd, u32 tile, int wv)
{
    return share_of(load_runs(p, bd, tile, wv));
}

__device__ __forceinline__ u32 share_at(const Share &s, u32 j)
{
    const u32 d1 = s.d1, d2 = s.d2, d3 = s.d3;
    return s.o0 + j + (j >= s.p1 ? d1 : 0u) + (j >= s.p2 ? d2 : 0u) + (j >= s.p3 ? d3 : 0u);
}

__device__ __forceinline__ u32 slot_hash(u64 rest)
{
    return ((u32)rest * 0x9e3779b1u + (u32)(rest >> 32) * 0x85ebca6bu) >> 23; // BW_SLOTS = 2^9
}

// the terms of a share of at most BW_CAP, in registers (so that the loads of
// the next share run while this one is worked on)
// (scalars: an array of HIP's vector type would be left in scratch memory)
template <typename AT> struct Staged {
    u64 k[BW_ROUNDS];
    typename Scalar<AT>::T x[BW_ROUNDS], y[BW_ROUNDS];
};

template <typename AT>
__device__ __forceinline__ void stage_load(Staged<AT> &r, const Share &t, const u64 *__restrict__ keys,
                                           const AT *__restrict__ amps)
{
    const u32 lane = (u32)sts_lane();
#pragma unroll
    for (int i = 0; i < BW_ROUNDS; ++i) {
        const u32 j = (u32)i * 64 + lane;
        if (j < t.n) {
            const u32 at = share_at(t, j);
            r.k[i] = keys[at];
            const AT a = amps[at];
            r.x[i] = a.x;
            r.y[i] = a.y;
        }
    }
}

template <typename AT> __device__ __forceinline__ void stage_store(WaveSmem<AT> &s, const Staged<AT> &r, u32 n)
{
    const u32 lane = (u32)sts_lane();
#pragma unroll
    for (int i = 0; i < BW_ROUNDS; ++i) {
        const u32 j = (u32)i * 64 + lane;
        if (j < n) {
            s.key[j] = r.k[i];
            AT a;
            a.x = r.x[i];
            a.y = r.y[i];
            s.amp[j] = a;
        }
    }
}

// stage the terms whose second hash has the prefix `pre` of `depth` bits;
// returns how many there are (more than BW_CAP: not all staged)
template <typename AT>
__device__ __forceinline__ u32 stage_part(WaveSmem<AT> &s, const Share &t, const u64 *__restrict__ keys,
                                       const AT *__restrict__ amps, u64 notmask, int depth, u64 pre)
{
    const u32 lane = (u32)sts_lane();
    u32 count = 0;
    for (u32 j0 = 0; j0 < t.n && count <= BW_CAP; j0 += 64) {
        const u32 j = j0 + lane;
        bool keep = false;
        u64 k = 0;
        u32 at = 0;
        if (j < t.n) {
            at = share_at(t, j);
            k = keys[at];
            keep = (sts_mix64(k & notmask) >> (64 - depth)) == pre;
        }
        const u64 m = wballot(keep);
        const u32 pos = count + sts_lanes_below(m);
        if (keep && pos < BW_CAP) {
            s.key[pos] = k;
            s.amp[pos] = amps[at];
        }
        count += (u32)__popcll(m);
    }
    return count;
}

// Group the `cnt` staged terms. Most groups have one member, whose outputs are
// one column of U each: those are listed (by staged index) from the front of
// s.lead; the others from its end, by the slot that holds their member list.
// First every slot counts the terms that hash to it and adds up their
// indices. A term alone in its slot is a group of one; of two terms in a slot
// each finds the other from the sum, and they are one group or two; only the
// terms of fuller slots (a tenth of them at half load) are left to open
// addressing on the masked key, all in one round as a rule.
template <typename AT, int M>
__device__ __forceinline__ void build_groups(WaveSmem<AT> &s, const GateLoc<M> &g, u32 cnt, u32 &singles, u32 &multis)
{
    const u32 lane = (u32)sts_lane();
    const u64 nm = g.nm;
    u64 key[BW_ROUNDS], other[BW_ROUNDS];
    u32 sl[BW_ROUNDS], sum[BW_ROUNDS], mate[BW_ROUNDS];
    u32 hard = 0; // a bit per round
    auto word = [&](u32 j, u64 k) { return (unsigned long long)(j + 1) << (16 * pattern_of<M>(g, k)); };
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        if (j < cnt) key[r] = s.key[j];
    }
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        if (j < cnt) {
            sl[r] = slot_hash(key[r] & nm);
            // indices below 2^9: the sum over all terms stays below 2^16
            atomicAdd(reinterpret_cast<u32 *>(&s.slot[sl[r]]), 0x10000u + j);
        }
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        sum[r] = 0;
        if (j < cnt) sum[r] = *reinterpret_cast<const u32 *>(&s.slot[sl[r]]);
    }
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        mate[r] = (sum[r] >> 16) == 2 ? (sum[r] & 0xffffu) - j : j;
        if (j < cnt) other[r] = s.key[mate[r]];
    }
    wave_sync();
    singles = 0;
    multis = 0;
    u32 nhard = 0;
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        const bool has = j < cnt;
        const bool pair = has && mate[r] != j && ((other[r] ^ key[r]) & nm) == 0;
        const bool one = has && !pair && sum[r] < 0x30000u;
        const bool left = has && sum[r] >= 0x30000u;
        const bool lead = pair && j < mate[r];
        if (has && !pair) s.slot[sl[r]] = 0;
        if (lead) s.slot[sl[r]] = word(j, key[r]) | word(mate[r], other[r]);
        const u64 m1 = wballot(one), m2 = wballot(lead), m3 = wballot(left);
        if (one) s.lead[singles + sts_lanes_below(m1)] = (unsigned short)j;
        if (lead) s.lead[BW_CAP - 1 - multis - sts_lanes_below(m2)] = (unsigned short)sl[r];
        if (m3) { // uniform
            const u32 at = nhard + sts_lanes_below(m3);
            if (left && at < 64) s.hard[at] = (unsigned short)j;
            hard |= left ? 1u << r : 0u;
        }
        singles += (u32)__popcll(m1);
        multis += (u32)__popcll(m2);
        nhard += (u32)__popcll(m3);
    }
    wave_sync();
    // open addressing for term j (when todo), true if it opened its group
    auto probe = [&](bool todo, u32 j, u64 k, u32 &at) {
        const u64 rest = k & nm;
        const unsigned long long mine = word(j, k);
        bool opened = false;
        at = slot_hash(rest);
        while (wballot(todo)) {
            if (todo) {
                const unsigned long long old = atomicCAS(&s.slot[at], 0ull, mine);
                if (old == 0) {
                    opened = true;
                    todo = false;
                } else { // any member tells the group
                    const int f = (__ffsll((long long)old) - 1) & ~15;
                    if ((s.key[(u32)((old >> f) & 0xffffu) - 1u] & nm) == rest) {
                        atomicOr(&s.slot[at], mine);
                        todo = false;
                    } else {
                        at = (at + 1) & (BW_SLOTS - 1);
                    }
                }
            }
        }
        return opened;
    };
    if (nhard && nhard <= 64) {
        const bool has = lane < nhard;
        const u32 j = has ? s.hard[lane] : 0u;
        u32 at;
        const bool opened = probe(has, j, s.key[j], at);
        wave_sync();
        bool one = false;
        if (opened) {
            const unsigned long long w = s.slot[at];
            one = (w & ~(0xffffull << ((__ffsll((long long)w) - 1) & ~15))) == 0;
            if (one) s.slot[at] = 0;
        }
        const u64 m1 = wballot(one), m2 = wballot(opened && !one);
        if (one) s.lead[singles + sts_lanes_below(m1)] = (unsigned short)j;
        if (opened && !one) s.lead[BW_CAP - 1 - multis - sts_lanes_below(m2)] = (unsigned short)at;
        singles += (u32)__popcll(m1);
        multis += (u32)__popcll(m2);
    } else if (nhard) { // many groups of several members: every group goes by its slot
#pragma unroll 1
        for (u32 r = 0; r < BW_ROUNDS; ++r) {
            const bool has = (hard >> r) & 1u;
            const u32 j = has ? r * 64 + lane : 0u;
            u32 at;
            const bool opened = probe(has, j, s.key[j], at);
            const u64 m = wballot(opened);
            if (opened) s.lead[BW_CAP - 1 - multis - sts_lanes_below(m)] = (unsigned short)at;
            multis += (u32)__popcll(m);
        }
    }
    wave_sync();
}

// body(ox, oy, rest, active) for the groups of a share, one per lane: the new
// amplitudes of its 2^M patterns (zeros in lanes without a group) and the key
// bits outside the gate; every lane of the wave takes part
// (grouped() runs between the grouping and the first call of body)
template <typename AT, int M, typename F, typename H>
__device__ __forceinline__ void staged_groups(WaveSmem<AT> &s, const AT *ucol, const GateLoc<M> &g, u32 cnt,
                                              H &&grouped, F &&body)
{
    typedef typename Scalar<AT>::T R;
    const u32 lane = (u32)sts_lane();
    u32 singles, multis;
    build_groups<AT, M>(s, g, cnt, singles, multis);
    grouped();
    const u32 rs = (singles + 63) >> 6, rm = (multis + 63) >> 6;
#pragma unroll 1
    for (u32 r = 0; r < rs + rm; ++r) {
        R ox[1 << M], oy[1 << M];
        u64 rest = 0;
        bool active;
        if (r < rs) {
            const u32 q = r * 64 + lane;
            active = q < singles;
            AT a;
            a.x = 0;
            a.y = 0;
            u32 j = 0;
            if (active) {
                const u32 i = s.lead[q];
                const u64 key = s.key[i];
                a = s.amp[i];
                rest = key & g.nm;
                j = pattern_of<M>(g, key);
            }
            const AT *col = ucol + ((1 << M) * j);
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT u = col[i];
                if constexpr (sizeof(R) == 4) { // the dense product's terms that are not zero
                    ox[i] = __builtin_fmaf(-u.y, a.y, u.x * a.x);
                    oy[i] = __builtin_fmaf(u.y, a.x, u.x * a.y);
                } else {
                    ox[i] = (R)0 + (u.x * a.x - u.y * a.y);
                    oy[i] = (R)0 + (u.x * a.y + u.y * a.x);
                }
            }
        } else {
            const u32 q = (r - rs) * 64 + lane;
            active = q < multis;
            u32 present = 0;
            R vx[1 << M], vy[1 << M];
#pragma unroll
            for (int j = 0; j < (1 << M); ++j) {
                vx[j] = 0;
                vy[j] = 0;
            }
            if (active) {
                const u32 sl = s.lead[BW_CAP - 1 - q];
                const unsigned long long w = s.slot[sl];
                s.slot[sl] = 0;
                const int f = (__ffsll((long long)w) - 1) & ~15;
                rest = s.key[(u32)((w >> f) & 0xffffu) - 1u] & g.nm;
#pragma unroll
                for (int j = 0; j < (1 << M); ++j) {
                    const u32 i = (u32)((w >> (16 * j)) & 0xffffu);
                    if (i) {
                        const AT a = s.amp[i - 1];
                        vx[j] = a.x;
                        vy[j] = a.y;
                        present |= 1u << j;
                    }
                }
            }
            // the product of group_out, with U from LDS (the same address in
            // every lane)
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                R ar = 0, ai = 0;
#pragma unroll
                for (int j = 0; j < (1 << M); ++j) {
                    const AT u = ucol[(1 << M) * j + i];
                    if constexpr (sizeof(R) == 4) {
                        ar = __builtin_fmaf(u.x, vx[j], ar);
                        ar = __builtin_fmaf(-u.y, vy[j], ar);
                        ai = __builtin_fmaf(u.x, vy[j], ai);
                        ai = __builtin_fmaf(u.y, vx[j], ai);
                    } else {
                        const R nr = ar + (u.x * vx[j] - u.y * vy[j]);
                        const R ni = ai + (u.x * vy[j] + u.y * vx[j]);
                        const bool has = (present >> j) & 1u;
                        ar = has ? nr : ar;
                        ai = has ? ni : ai;
                    }
                }
                ox[i] = ar;
                oy[i] = ai;
            }
        }
        body(ox, oy, rest, active);
    }
    wave_sync();
}

// the groups of a share: of at most BW_CAP terms, already staged; a larger one
// is staged here in parts
// (grouped() runs once, after the first grouping)
template <typename AT, int M, typename F, typename H>
__device__ __forceinline__ void share_parts(WaveSmem<AT> &s, const AT *ucol, const GateLoc<M> &g, const Share &t,
                                            const u64 *__restrict__ keys, const AT *__restrict__ amps, H &&grouped,
                                            F &&body)
{
    bool first = true;
    PartWalk part;
    part.begin(t.n, BW_CAP);
    do {
        u32 cnt = t.n;
        if (part.depth) {
            cnt = uni(stage_part<AT>(s, t, keys, amps, g.nm, part.depth, part.pre));
            while (cnt > BW_CAP) {
                part.split();
                cnt = uni(stage_part<AT>(s, t, keys, amps, g.nm, part.depth, part.pre));
            }
        }
        wave_sync();
        staged_groups<AT, M>(s, ucol, g, cnt, [&]() {
            if (first) grouped();
            first = false;
        }, body);
    } while (part.next());
}

template <typename AT, int M, typename F>
__device__ __forceinline__ void share_groups(WaveSmem<AT> &s, const AT *ucol, const GateLoc<M> &g, const Share &t,
                                             const u64 *__restrict__ keys, const AT *__restrict__ amps, F &&body)
{
    if (t.n == 0) return;
    if (t.n <= BW_CAP) {
        Staged<AT> st;
        stage_load<AT>(st, t, keys, amps);
        stage_store<AT>(s, st, t.n);
    }
    share_parts<AT, M>(s, ucol, g, t, keys, amps, []() {}, body);
}

// before the first share (the caller's barrier follows); called by the first
// NW waves, or by all of a larger workgroup
template <typename AT, int M, int NW>
__device__ __forceinline__ void smem_begin(BktSmem<AT, NW> &s, const GateArg &g)
{
    typedef typename Scalar<AT>::T R;
    if (threadIdx.x < NW * 64) {
        WaveSmem<AT> &w = s.w[threadIdx.x >> 6];
        for (int i = sts_lane(); i < BW_SLOTS; i += 64) w.slot[i] = 0;
    }
    if (threadIdx.x < (1 << (2 * M))) {
        const int i = (int)threadIdx.x & ((1 << M) - 1), j = (int)threadIdx.x >> M;
        AT u;
        u.x = UEntry<R, M>::re(g, i, j);
        u.y = UEntry<R, M>::im(g, i, j);
        s.ucol[threadIdx.x] = u;
    }
}

__device__ __forceinline__ u32 bkt_tiles(const BktPlan &p) { return 1u << (p.hb - STS_BKT_DIMS); }

// candidates of one output pattern, one per lane, to the wave's slab: the
// window's from its start, those above it from its end
struct SlabOut {
    u32 c_in, c_ab, c_all; // the wave's claims so far, and its candidates (the same in every lane)
    bool fits;
};

template <typename AT>
__device__ __forceinline__ void slab_put(SlabOut &o, u64 *sk, u64 *sw, AT *sa, u32 room, bool inw, bool ab, u64 key,
                                         u64 wb, const AT &v)
{
    const u64 m_ab = wballot(ab), m_in = wballot(inw);
    const u32 n_ab = (u32)__popcll(m_ab), n_in = (u32)__popcll(m_in);
    o.fits = o.fits && o.c_in + o.c_ab + n_ab + n_in <= room;
    if (o.fits && (inw || ab)) {
        const u32 at = inw ? o.c_in + sts_lanes_below(m_in) : room - 1u - o.c_ab - sts_lanes_below(m_ab);
        sts_store_at(sk, at * 8u, key);
        sts_store_at(sa, at * (u32)sizeof(AT), v);
        if (inw) sts_store_at(sw, at * 8u, wb);
    }
    o.c_in += n_in;
    o.c_ab += n_ab;
}

// the gate that a step's first kernel was given, into device memory
__device__ __forceinline__ void put_gate(const GateArg &g, GateArg *dst)
{
    const u32 *src = reinterpret_cast<const u32 *>(&g);
    u32 *d = reinterpret_cast<u32 *>(dst);
    for (u32 i = threadIdx.x; i < sizeof(GateArg) / sizeof(u32); i += STS_WG) d[i] = src[i];
}

// a candidate's weight to the exponent bins
__device__ __forceinline__ void bin_weight(const PassBufs &b, u64 *s_hi, u64 *s_lo, int hot_lo, u64 wb, bool direct)
{
    const int e = (int)(wb >> 52);
    const u64 mant = sts_mant(wb);
    const int bin = e - TT_EBASE, hd = e - hot_lo;
    if (!direct && ((unsigned)hd < (unsigned)TT_HOT || (unsigned)bin < (unsigned)TT_NB)) {
        const int f2 = (int)((wb >> 50) & (TT_HSUB - 1)), copy = (int)(threadIdx.x % TT_HCOPIES);
        const int slot = (unsigned)hd < (unsigned)TT_HOT ? TT_NB + (hd * TT_HSUB + f2) * TT_HCOPIES + copy : bin;
        atomicAdd(&s_hi[slot], mant >> 26);
        atomicAdd(&s_lo[slot], (mant & ((1ull << 26) - 1)) | (1ull << 44));
    } else {
        atomicAdd(&b.h1[e], 1ull);
        atomicAdd(&b.h1[STS_NBIN + e], mant >> 26);
        atomicAdd(&b.h1[2 * STS_NBIN + e], mant & ((1ull << 26) - 1));
    }
}

// lower exponent field of the two octaves a small step's slabs hold: the
// previous cut's and the one its threshold lies nearer to
__device__ __forceinline__ int small_window(const DevCtl *ctl)
{
    const int e = ctl->e_pred;
    return e > 0 && !((ctl->thr_wbits >> 51) & 1ull) ? e - 1 : e;
}

// ---------------------------------------------------------------------------
// histogram pass: exponent histogram with exact mantissa sums of all new
// weights (persistent grid). With b.recover it runs only after a sampled
// window that missed (or where nothing can be cut, b.whole), and its last
// workgroup does the level-1 pick. With b.keep it also puts the candidates (those
// from slab_floor on), with their weights, into the share's slab, from which the
// following passes then read: none of them multiplies again unless a slab was too
// small or the cut lies lower. The pick's tables take the place of the waves' (two
// workgroups per CU instead of one).
// ---------------------------------------------------------------------------
template <typename AT> union HistSmem {
    struct {
        BktSmem<AT, BW> s;
        u64 hi[TT_SLOTS], lo[TT_SLOTS];
    } pass;
    sts_select::Level1Smem<STS_WG> l1;
};

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_hist(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ HistSmem<AT> u;
    __shared__ u32 s_flag;
    BktSmem<AT, BW> &s = u.pass.s;
    u64 *const s_hi = u.pass.hi, *const s_lo = u.pass.lo;
    DevCtl *ctl = b.ctl;
    if (b.recover && !b.whole && !ctl->need_full) return; // uniform
    smem_begin<AT, M, BW>(s, g);
    for (int i = threadIdx.x; i < TT_SLOTS; i += STS_WG) {
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
    const u32 ntiles = bkt_tiles(g.bkt);
    const int e_prev = ctl->e_pred;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int hot_lo = (e_prev >= 0 ? e_prev : TT_EBASE + 116) - (TT_HOT - 4);
    const int shift = b.slab_shift, e_floor = slab_floor(b, e_prev);
    if (b.keep && blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->side_dense = 0;
        ctl->side_ntiles = (u64)ntiles << 2;
        ctl->side_slab_shift = shift;
        ctl->side_spt_log2 = 2;
    }
    __syncthreads();
    int since_flush = 0;
    // the runs of 16 shares are loaded together (a state far below its size bound
    // has many empty ones, each of which would wait for a load: 92 us for 65,536
    // of them)
    uint2 next = make_uint2(0, 0);
    int held = 0;
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (since_flush == BW_FLUSH) {
            // a tile adds at most 4 * BW_BINNED * 4 candidates to the bins
            __syncthreads();
            flush_bins(b, s_hi, s_lo, hot_lo);
            since_flush = 0;
            __syncthreads();
        }
        ++since_flush;
        if ((held & 15) == 0) {
            const u32 t = tile + ((u32)sts_lane() >> 2) * gridDim.x;
            next = load_runs(g.bkt, b.bd_in, t < ntiles ? t : 0u, wv);
        }
        const Share sh = share_of(next, 4 * (held++ & 15));
        const bool direct = sh.n > BW_BINNED;
        const u32 sl = (tile << 2) + (u32)wv;
        const u64 slab = (u64)sl << shift;
        SlabOut so = {0, 0, 0, true};
        share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, b.keys, (const AT *)b.amps,
                            [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                const bool cand = active && nonzero(o);
                const u64 wb = weight_bits(o);
                if (cand) bin_weight(b, s_hi, s_lo, hot_lo, wb, direct);
                so.c_all += (u32)__popcll(wballot(cand));
                if (b.keep) // uniform
                    slab_put<AT>(so, b.side_key + slab, b.side_w + slab, (AT *)b.side_amp + slab, 1u << shift,
                                 cand && (int)(wb >> 52) >= e_floor, false,
                                 rest | pattern_bits<M>(gl, i), wb, o);
            }
        });
        if (sts_lane() == 0) {
            b.w_all[sl] = so.c_all;
            if (b.keep) {
                b.t_above[sl] = 0;
                b.t_side[sl] = so.c_in;
                if (!so.fits) atomicOr(&ctl->w_over, 1u);
            }
        }
    }
    __syncthreads();
    flush_bins(b, s_hi, s_lo, hot_lo);
    if (!b.recover || !sts_last_block(&ctl->done[0], &s_flag)) return;
    sts_select::pick_level1<STS_WG>(b, 0, 0, 3, u.l1, sts_select::DeviceBins<STS_WG>{b.h1});
}

// ---------------------------------------------------------------------------
// weighing pass of a sampled step (large states): the window [w_lo, w_hi] is
// set, so the exact masses needed are only the total's, the mass above the
// window and the window's own level-2 bins. The first two are summed in
// registers: a weight of the exponent fields [L, L + FINE_EXPS), L <= e_w, is a
// multiple of u = 2^(L - 1075) below 2^80 u, and is split exactly into a
// multiple of 2^40 u (by adding and subtracting 1.5 * 2^92 u) and a rest of
// at most 2^39 u; sums of up to 2^12 of either stay exact in binary64. Weights
// of other exponents go to the exponent bins.
// ---------------------------------------------------------------------------
struct FineSums {
    double t1, t2, a1, a2; // total and above the window: the two parts
};

// add a lane's sums to the workgroup's (LDS, two's complement) and clear them
__device__ __forceinline__ void flush_fine(u64 *s_acc, FineSums &f, double k1, double k2)
{
    const double v[4] = {f.t1 * k1, f.t2 * k2, f.a1 * k1, f.a2 * k2};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (v[i] != 0.0) atomicAdd(&s_acc[i], (u64)(long long)v[i]);
    f.t1 = f.t2 = f.a1 = f.a2 = 0.0;
}

// One workgroup per CU, whose waves' tables fill the LDS (16 waves for
// complex64, 12 for complex128): the pass waits on chains of LDS round trips,
// and more waves hide more of them. Four waves have one tile. Bound by vector
// instructions (about 1730 a wave and share of 256 terms, 59% of its time):
// 313 us at 2^24 complex64 terms, where the sorted path took 345 for its three
// scatters, 83 for their counts and 321 for the histogram. (With 12 waves and
// no register spills 341 when it took 323.)
template <typename AT> struct WeighWaves {
    static constexpr int value = sizeof(AT) == 8 ? 16 : 12;
};
constexpr int FINE_EXPS = 28; // exponent fields that the registers sum, from L
// LDS bins for the rest of [TT_EBASE, TT_EBASE + TT_NB), the histogram pass's
// range. (Bins in device memory, where every workgroup adds to the same few words,
// took 5300 us at 2^20 terms whose cut lies 2^16 below most weights, and LDS bins
// 245; those from L - 38 to L + 25 only, 2800 us where small weights lie lower.)
constexpr int WEIGH_COLD = TT_NB - FINE_EXPS;
// Most rounds of 64 groups that a share may take: one of BW_BINNED terms in
// parts of usual size takes at most some 30, one in many small parts more, and
// is left to the histogram pass. A lane's sums then stay exact between flushes.
constexpr u32 WEIGH_ROUNDS = 64;
static_assert(WEIGH_ROUNDS * BW_FLUSH * 4 <= 1 << 12, "four weights a round, sums of up to 2^12 of them");

template <typename AT, int M>
__global__ void __launch_bounds__(64 * WeighWaves<AT>::value, 1)
    k_bkt_weigh(const GateArg *__restrict__ gp, PassBufs b)
{
    constexpr int NW = WeighWaves<AT>::value, NT = NW * 64, TPW = NW / 4;
    const GateArg &g = *gp;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, NW> s;
    __shared__ u64 s_hi[WEIGH_COLD], s_lo[WEIGH_COLD]; // sums of mantissa >> 20; & (2^20 - 1), plus count << 44
    __shared__ u64 s_w2[TT_W2]; // level-2 bins of the window: sums of the 41 mantissa bits below the bin's,
    __shared__ u32 s_w2c[TT_W2]; // and counts
    __shared__ u64 s_acc[7]; // flush_fine's four sums, then candidates: all, above the window, inside it
    DevCtl *ctl = b.ctl;
    if (!ctl->w_mode) return; // uniform: no window; the recovering histogram pass does the step
    smem_begin<AT, M, NW>(s, g);
    for (int i = threadIdx.x; i < WEIGH_COLD; i += NT) {
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
    for (int i = threadIdx.x; i < TT_W2; i += NT) {
        s_w2[i] = 0;
        s_w2c[i] = 0;
    }
    if (threadIdx.x < 7) s_acc[threadIdx.x] = 0;
    const u64 *keys = b.keys;
    const AT *amps = (const AT *)b.amps;
    const u32 ntiles = bkt_tiles(g.bkt);
    const u64 w_lo = ctl->w_lo, w_hi = ctl->w_hi;
    const u32 d_lo = uni((u32)((((1ull << 52) - 1) - (w_hi & ((1ull << 52) - 1))) >> 41));
    const u32 d_top = 2047u - d_lo;
    // the window's edges are multiples of 2^47 in the weight bits: the high
    // words decide
    const u32 wL = uni((u32)(w_lo >> 32)), wH = uni((u32)((w_hi + 1) >> 32));
    const int L = (int)uni((u32)ctl->w_L);
    const u32 rL = (u32)L << 20, rN = (u32)FINE_EXPS << 20;
    const double C = __longlong_as_double((long long)(((u64)(L + 40) << 52) | (1ull << 51)));
    const double k1 = __longlong_as_double((long long)((u64)(2058 - L) << 52));
    const double k2 = __longlong_as_double((long long)((u64)(2098 - L) << 52));
    FineSums f = {0.0, 0.0, 0.0, 0.0};
    u64 n_all = 0, n_above = 0, n_win = 0; // the wave's totals (the same in every lane)
    bool over = false;
    const int shift = b.slab_shift;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->side_dense = 0;
        ctl->side_ntiles = (u64)ntiles << 2;
        ctl->side_slab_shift = shift;
        ctl->side_spt_log2 = 2;
    }
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tw = wv & 3; // the wave's share of its tile
    auto flush = [&]() {
        flush_fine(s_acc, f, k1, k2);
        for (int i = threadIdx.x; i < WEIGH_COLD; i += NT) {
            const u64 lo = s_lo[i];
            if (lo >> 44) {
                const u128 tot = ((u128)s_hi[i] << 20) + (u128)(lo & ((1ull << 44) - 1));
                const int e = TT_EBASE + i + (TT_EBASE + i < L ? 0 : FINE_EXPS);
                atomicAdd(&b.h1[e], lo >> 44);
                atomicAdd(&b.h1[STS_NBIN + e], (u64)(tot >> 26));
                atomicAdd(&b.h1[2 * STS_NBIN + e], (u64)tot & ((1ull << 26) - 1));
            }
            s_hi[i] = 0;
            s_lo[i] = 0;
        }
        for (int i = threadIdx.x; i < TT_W2; i += NT) {
            const u32 c = s_w2c[i];
            if (c) {
                const u32 d = d_lo + (u32)i;
                // the bits a bin's mantissas share: the leading one and its top fraction bits
                const u64 top = ((u64)(2048u | (2047u - d)) << 41);
                const u128 tot = (u128)top * c + (u128)s_w2[i];
                atomicAdd(&b.h2w[d], (u64)c);
                atomicAdd(&b.h2w[STS_NBIN + d], (u64)(tot >> 26));
                atomicAdd(&b.h2w[2 * STS_NBIN + d], (u64)tot & ((1ull << 26) - 1));
            }
            s_w2[i] = 0;
            s_w2c[i] = 0;
        }
    };
    __syncthreads();
    // tiles in flight: the terms of this wave's next share are loaded while
    // the current one is worked on, and the runs of the one after that
    const u32 step = gridDim.x * TPW;
    u32 tile = blockIdx.x * TPW + (u32)(wv >> 2);
    const u32 rounds = (ntiles + step - 1) / step; // the same for every wave: the flushes have barriers
    auto runs = [&](u32 t) { return load_runs(g.bkt, b.bd_in, t < ntiles ? t : 0u, tw); };
    Share nx = share_of(runs(tile));
    if (tile >= ntiles) nx.n = 0;
    Staged<AT> st;
    if (nx.n <= BW_CAP) stage_load<AT>(st, nx, keys, amps);
    uint2 d2 = runs(tile + step);
    for (u32 it = 0; it < rounds; ++it, tile += step) {
        if (it && it % BW_FLUSH == 0) {
            // a lane has added at most BW_FLUSH * WEIGH_ROUNDS * 4 weights (or
            // the sums are not used), and the bins at most 16 * 16 * BW_BINNED * 4
            __syncthreads();
            flush();
            __syncthreads();
        }
        const Share sh = nx;
        if (sh.n <= BW_CAP) stage_store<AT>(s.w[wv], st, sh.n);
        if (tile >= ntiles) continue;
        const u32 sl = (tile << 2) + (u32)tw;
        const u64 slab = (u64)sl << shift;
        u64 *const sk = b.side_key + slab;
        u64 *const sw = b.side_w + slab;
        AT *const sa = (AT *)b.side_amp + slab;
        const u32 room = 1u << shift;
        u32 c_in = 0, c_ab = 0, c_all = 0; // the wave's claims so far (the same in every lane)
        bool fits = true;
        auto advance = [&]() {
            nx = share_of(d2);
            if (tile + step >= ntiles) nx.n = 0;
            if (nx.n <= BW_CAP) stage_load<AT>(st, nx, keys, amps);
            d2 = runs(tile + 2 * step);
        };
        if (sh.n > BW_BINNED) { // more than the sums are bounded for: the histogram pass takes the step
            over = true;
            advance();
            continue;
        }
        u32 taken = 0;
        share_parts<AT, M>(s.w[wv], s.ucol, gl, sh, keys, amps, advance, [&](const auto &ox, const auto &oy, u64 rest, bool active) {
            ++taken;
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                const u64 wb = weight_bits(o); // 0 in lanes without a group
                const u32 hw = (u32)(wb >> 32);
                // (a complex64 weight is zero only when both parts are)
                const bool cand = sizeof(AT) == 8 ? wb != 0 : nonzero(o);
                const bool ab = hw >= wH, inw = hw >= wL && !ab;
                const u64 m_ab = wballot(ab), m_in = wballot(inw), m_c = wballot(cand);
                const u64 m_far = m_c & wballot(hw - rL >= rN);
                double w = __longlong_as_double((long long)wb);
                if (m_far) { // uniform: some weights are too far from the window for the sums
                    if (cand && hw - rL >= rN) {
                        w = 0.0;
                        const int e_ = (int)(wb >> 52), bin = e_ - TT_EBASE - (e_ < L ? 0 : FINE_EXPS);
                        const u64 mant = sts_mant(wb);
                        if ((unsigned)bin < (unsigned)WEIGH_COLD) {
                            atomicAdd(&s_hi[bin], mant >> 20);
                            atomicAdd(&s_lo[bin], (mant & ((1ull << 20) - 1)) | (1ull << 44));
                        } else {
                            atomicAdd(&b.h1[e_], 1ull);
                            atomicAdd(&b.h1[STS_NBIN + e_], mant >> 26);
                            atomicAdd(&b.h1[2 * STS_NBIN + e_], mant & ((1ull << 26) - 1));
                        }
                    }
                }
                const double c1 = (w + C) - C, c2 = w - c1;
                const double one = ab ? 1.0 : 0.0;
                f.t1 += c1;
                f.t2 += c2;
                f.a1 = __builtin_fma(c1, one, f.a1);
                f.a2 = __builtin_fma(c2, one, f.a2);
                if (inw) {
                    const u32 rel = d_top - ((hw >> 9) & 2047u); // below TT_W2: three sub-bins of 1/32 octave
                    atomicAdd(&s_w2[rel], wb & ((1ull << 41) - 1));
                    atomicAdd(&s_w2c[rel], 1u);
                }
                c_all += (u32)__popcll(m_c);
                // to the slab: the window's from its start, those above it from its end
                const u32 n_ab = (u32)__popcll(m_ab), n_in = (u32)__popcll(m_in);
                fits = fits && c_in + c_ab + n_ab + n_in <= room;
                if (fits) {
                    const u64 key = rest | pattern_bits<M>(gl, i);
                    if (ab) {
                        const u32 at = (room - 1u - c_ab - sts_lanes_below(m_ab)) * 8u;
                        sts_store_at(sk, at, key);
                        sts_store_at(sa, at * (u32)(sizeof(AT) / 8), o);
                    }
                    if (inw) {
                        const u32 at = (c_in + sts_lanes_below(m_in)) * 8u;
                        sts_store_at(sk, at, key);
                        sts_store_at(sw, at, wb);
                        sts_store_at(sa, at * (u32)(sizeof(AT) / 8), o);
                    }
                }
                c_in += n_in;
                c_ab += n_ab;
            }
        });
        if (sts_lane() == 0) {
            b.w_all[sl] = c_all;
            b.t_above[sl] = c_ab;
            b.t_side[sl] = c_in;
        }
        if (!fits || taken > WEIGH_ROUNDS) over = true;
        n_all += c_all;
        n_above += c_ab;
        n_win += c_in;
    }
    if (sts_lane() == 0) {
        if (over) atomicOr(&ctl->w_over, 1u);
        atomicAdd(&s_acc[4], n_all);
        atomicAdd(&s_acc[5], n_above);
        atomicAdd(&s_acc[6], n_win);
    }
    __syncthreads();
    flush();
    __syncthreads();
    if (threadIdx.x < 7) b.wpart[threadIdx.x * STS_MAX_GROUPS + blockIdx.x] = s_acc[threadIdx.x];
}

// ---------------------------------------------------------------------------
// sampling pass (as k_tile_sample): the gate on evenly spaced tiles, one per
// workgroup, or on all of them for a fine window, which then holds the cut for
// certain (by count; by mass up to the rounding of its sums). A chain of
// latencies - a share's tables, bins to device memory, the last workgroup's
// scans: 24 us on the 512 tiles of 100,003 terms, 16 on 128 of them, 24 on 256
// tiles of 2^24 terms.
// (the gate comes by value and goes to device memory for the step's other
// kernels: a launch of its own for that cost 5 us a step)
// ---------------------------------------------------------------------------
// Sampled candidates in a window below which the step goes without one. As a rule a
// window has hundreds; where the cut lies in the tail of the kept weights and the
// window has a handful, it misses more often than not, which costs the weighing pass
// for nothing: rotations by 1e-4 at 2^24 terms 1270 us a step, without a window 1080.
// With 8 and more, windows that held the cut were lost (by 3e-3 800 us instead of 660).
constexpr u32 SAMPLE_LEAST = 4;

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_sample(GateArg g, PassBufs b)
{
    if (blockIdx.x == 0) put_gate(g, b.gate_dst);
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, BW> s;
    __shared__ SampleSmem ss;
    DevCtl *ctl = b.ctl;
    const int e_prev = ctl->e_pred;
    if (e_prev < 0) return; // uniform: nothing to centre the bins on
    smem_begin<AT, M, BW>(s, g);
    SampleAcc acc;
    sample_begin(ss, acc, ctl);
    __syncthreads();
    const u32 ntiles = bkt_tiles(g.bkt);
    const u32 stride = ntiles > gridDim.x ? ntiles / gridDim.x : 1;
    const u32 tile = blockIdx.x * stride;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int e_lo = e_prev - STS_SW_EXPS / 2;
    u32 seen = 0;
    if (tile < ntiles) {
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        if (sh.n <= BW_CAP) { // an overfull share is left out of the sample
            seen = sh.n;
            share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, b.keys, (const AT *)b.amps, [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
                for (int i = 0; i < (1 << M); ++i) {
                    AT o;
                    o.x = ox[i];
                    o.y = oy[i];
                    if (active && nonzero(o)) sample_add(ss, acc, weight_bits(o), e_lo);
                }
            });
        }
    }
    sample_flush(ss, acc, b, sts_lane() == 0 ? seen : 0u);
    if (!sts_last_block(&ctl->done[2], &ss.flag)) return;
    sample_finish(ss, b, e_lo, *b.n_in, b.fine_window, SAMPLE_LEAST);
}

// ---------------------------------------------------------------------------
// the passes of a step whose window missed the cut (they exit at once when it
// held it): the level-2 bins of the cut's exponent, picked by the last workgroup;
// and the survivors per share. Both read the weights in the slabs; where a slab
// was too small for its candidates, these are computed again and those of the
// cut's exponent go to the side buffer, densely packed (one claim per tile).
// A gate without a truncation has the count only, which puts the new terms into
// the slabs for the copy (347 us at 2^22 complex64 terms when they were computed
// three times, 251 with the sort)
// ---------------------------------------------------------------------------
// the entries of a wave's slabs, one tile after the other: the counts of 64 tiles
// are loaded together
struct SlabCounts {
    u32 held = 0, c = 0;
    __device__ __forceinline__ u32 next(const PassBufs &b, u32 tile, u32 ntiles, int wv)
    {
        if ((held & 63u) == 0) {
            const u32 t = tile + (u32)sts_lane() * gridDim.x;
            c = t < ntiles ? b.t_side[(t << 2) + (u32)wv] : 0u;
        }
        return (u32)__builtin_amdgcn_readlane((int)c, (int)(held++ & 63u));
    }
};

// f(weight, index) of the n entries of a slab, a wave's loads in flight together
template <typename F> __device__ __forceinline__ void slab_weights(const u64 *__restrict__ w, u32 n, F &&f)
{
    constexpr int UN = 8;
    for (u32 i0 = (u32)sts_lane(); i0 < n; i0 += 64 * UN) {
        u64 x[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) x[r] = i0 + 64u * (u32)r < n ? w[i0 + 64u * (u32)r] : ~0ull;
#pragma unroll
        for (int r = 0; r < UN; ++r)
            if (x[r] != ~0ull) f(x[r], i0 + 64u * (u32)r); // (no weight has all bits set)
    }
}

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_extract(const GateArg *__restrict__ gp, PassBufs b)
{
    using namespace sts_select;
    const GateArg &g = *gp;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, BW> s;
    __shared__ u32 s_cnt[BW];
    __shared__ u64 s_base;
    __shared__ u64 s_low[STS_NBIN]; // sums of the 41 mantissa bits below the bin's, and counts
    __shared__ u32 s_num[STS_NBIN];
    __shared__ CutSmem s_cut;
    __shared__ Sub s_sub;
    __shared__ u32 s_flag;
    DevCtl *ctl = b.ctl;
    if (ctl->pred_hit || ctl->keep_all) return; // uniform
    smem_begin<AT, M, BW>(s, g);
    for (int i = threadIdx.x; i < STS_NBIN; i += STS_WG) {
        s_low[i] = 0;
        s_num[i] = 0;
    }
    const int e_star = ctl->e_star;
    const u64 *keys = b.keys;
    const AT *amps = (const AT *)b.amps;
    const u32 ntiles = bkt_tiles(g.bkt);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool slabs = ctl->slab_all;
    auto flush = [&]() {
        for (int i = threadIdx.x; i < STS_NBIN; i += STS_WG) {
            const u32 c = s_num[i];
            if (!c) continue;
            const u128 tot = (u128)digit_mant((u32)i, e_star) * c + (u128)s_low[i];
            atomicAdd(&b.h2w[i], (u64)c);
            atomicAdd(&b.h2w[STS_NBIN + i], (u64)(tot >> 26));
            atomicAdd(&b.h2w[2 * STS_NBIN + i], (u64)tot & ((1ull << 26) - 1));
            s_low[i] = 0;
            s_num[i] = 0;
        }
    };
    __syncthreads();
    u32 since = 0;
    SlabCounts counts;
    for (u32 tile = blockIdx.x; slabs && tile < ntiles; tile += gridDim.x) {
        if (++since > 1u << 8) { // (a tile has four slabs of at most 2^12 entries: sums stay below 2^64)
            __syncthreads();
            flush();
            since = 1;
            __syncthreads();
        }
        const u32 sl = (tile << 2) + (u32)wv;
        slab_weights(b.side_w + ((u64)sl << b.slab_shift), counts.next(b, tile, ntiles, wv), [&](u64 w, u32) {
            if ((int)(w >> 52) != e_star) return;
            const u32 d = 2047u - ((u32)(w >> 41) & 2047u);
            atomicAdd(&s_low[d], w & LOW41);
            atomicAdd(&s_num[d], 1u);
        });
    }
    if (slabs) {
        __syncthreads();
        flush();
    }
    for (u32 tile = blockIdx.x; !slabs && tile < ntiles; tile += gridDim.x) {
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        u32 cnt = 0;
        share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, keys, amps, [&](const auto &ox, const auto &oy, u64, bool active) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                cnt += (u32)__popcll(wballot(active && nonzero(o) && (int)(weight_bits(o) >> 52) == e_star));
            }
        });
        if (sts_lane() == 0) s_cnt[wv] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) s_base = atomicAdd(&ctl->side_n, (u64)s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3]);
        __syncthreads();
        u64 at = s_base;
        for (int w = 0; w < wv; ++w) at += s_cnt[w];
        share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, keys, amps,
                            [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                const u64 wb = weight_bits(o);
                const bool take = active && nonzero(o) && (int)(wb >> 52) == e_star;
                const u64 m = wballot(take);
                const u64 p = at + sts_lanes_below(m);
                if (take && p < b.side_cap) {
                    b.side_key[p] = rest | pattern_bits<M>(gl, i);
                    b.side_w[p] = wb;
                    const u32 d = 2047u - ((u32)(wb >> 41) & 2047u);
                    const u64 mant = sts_mant(wb);
                    if (sh.n > (1u << 19)) { // more than a bin of the workgroup holds
                        atomicAdd(&b.h2w[d], 1ull);
                        atomicAdd(&b.h2w[STS_NBIN + d], mant >> 26);
                        atomicAdd(&b.h2w[2 * STS_NBIN + d], mant & ((1ull << 26) - 1));
                    } else {
                        atomicAdd(&s_low[d], mant & LOW41);
                        atomicAdd(&s_num[d], 1u);
                    }
                }
                at += (u64)__popcll(m);
            }
        });
        __syncthreads();
        flush();
    }
    if (!sts_last_block(&ctl->done[1], &s_flag)) return;
    if (threadIdx.x == 0) {
        s_sub.cnt_before = ctl->cnt_before;
        s_sub.mb = 0;
        s_sub.vpre = 0;
        s_sub.vshift = 116;
        s_sub.count = ctl->sub_count;
    }
    __syncthreads();
    const bool ok = pick_digit<STS_WG>(AgentBins{b.h2w}, ctl->K, make128(ctl->R_lo, ctl->R_hi), 11, &s_sub, s_cut.m,
                                       s_cut.c, &s_cut.hit);
    if (ok && threadIdx.x <= STS_SUB_REGIONS) st_agent(&b.sub_cnt[threadIdx.x * 32], 0u);
    if (threadIdx.x == 0) {
        if (ok) {
            sub_store(s_sub, ctl);
            ctl->level = 2;
        } else {
            atomicOr(&ctl->flags, STS_F_UNRESOLVED);
        }
    }
    for (int i = threadIdx.x; i < 3 * STS_NBIN; i += STS_WG) st_agent(&b.h2w[i], 0ull);
}

template <typename AT> __device__ __forceinline__ bool survives(u64 wb, u64 key, bool all, u64 thr_w, u64 thr_k)
{
    return all || wb > thr_w || (wb == thr_w && key <= thr_k);
}

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_count(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, BW> s;
    DevCtl *ctl = b.ctl;
    const bool all = b.materialise;
    if (!all && (ctl->pred_hit || ctl->keep_all)) return; // uniform
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const u32 ntiles = bkt_tiles(g.bkt);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (!all && ctl->slab_all) { // uniform
        SlabCounts counts;
        for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
            const u32 sl = (tile << 2) + (u32)wv;
            const u64 slab = (u64)sl << b.slab_shift;
            u32 cnt = 0;
            slab_weights(b.side_w + slab, counts.next(b, tile, ntiles, wv), [&](u64 w, u32 i) {
                cnt += w > thr_w || (w == thr_w && b.side_key[slab + i] <= thr_k) ? 1u : 0u;
            });
            cnt = wave_incl_scan(cnt);
            if (sts_lane() == 63) b.w_kept[sl] = cnt;
        }
        return;
    }
    smem_begin<AT, M, BW>(s, g);
    __syncthreads();
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        const u32 sl = (tile << 2) + (u32)wv;
        const u64 slab = (u64)sl << b.slab_shift;
        u32 cnt = 0;
        SlabOut so = {0, 0, 0, true};
        share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, b.keys, (const AT *)b.amps, [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                const u64 key = rest | pattern_bits<M>(gl, i);
                const bool take = active && nonzero(o) && survives<AT>(weight_bits(o), key, all, thr_w, thr_k);
                cnt += (u32)__popcll(wballot(take));
                if (all) // uniform
                    slab_put<AT>(so, b.side_key + slab, b.side_w + slab, (AT *)b.side_amp + slab, 1u << b.slab_shift, false,
                                 take, key, 0, o);
            }
        });
        if (sts_lane() == 0) {
            b.w_kept[sl] = cnt;
            if (all) {
                b.t_above[sl] = so.c_ab;
                b.t_side[sl] = 0;
                if (!so.fits) atomicOr(&ctl->w_over, 1u);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// write pass: a wave writes its share's survivors at its offset, bucket by
// bucket (4 << delta of them), and the output's bucket table
// ---------------------------------------------------------------------------
constexpr int BW_SUBS = 64; // output buckets of a share, at most 4 << 4

// rank of this lane's item among the wave's items of the same sub-bucket so
// far (cnt: the running counts, in LDS); lanes without one take part
__device__ __forceinline__ u32 sub_rank(bool keep, u32 sub, int bits, u32 *cnt)
{
    u64 peers = wballot(keep);
    for (int t = 0; t < bits; ++t) {
        const u64 bb = wballot((sub >> t) & 1u);
        peers &= ((sub >> t) & 1u) ? bb : ~bb;
    }
    u32 pre = 0;
    const u32 below = sts_lanes_below(peers);
    if (keep) pre = __hip_atomic_load(&cnt[sub], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
    if (keep && below == 0)
        __hip_atomic_store(&cnt[sub], pre + (u32)__popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
    return pre + below;
}

__device__ __forceinline__ u32 sub_bucket(const BktPlan &p, u64 key)
{
    u32 sub = sts_parity(key, p.cm[0]) | (sts_parity(key, p.cm[1]) << 1);
    for (int t = 0; t < p.delta; ++t) sub |= sts_parity(key, p.rm[t]) << (2 + t);
    return sub;
}

// turn the wave's sub-bucket counts into starts (from `base`) and write the
// output's bucket table
__device__ __forceinline__ void sub_starts(const BktPlan &p, const PassBufs &b, u32 tile, int wv, u32 base, u32 *cnt)
{
    const u32 lane = (u32)sts_lane();
    const u32 nsub = 4u << p.delta;
    // memory order: refinement bits above the coordinates
    const u32 c = lane < nsub ? __hip_atomic_load(&cnt[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
    const u32 beg = base + wave_incl_scan(c) - c;
    __builtin_amdgcn_wave_barrier();
    if (lane < nsub) {
        __hip_atomic_store(&cnt[lane], beg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const u32 in = bkt_rep(p, tile) ^ bkt_comb(p, (lane & 3u) | ((u32)wv << 2));
        b.bd_out[(in << p.delta) | (lane >> 2)] = make_uint2(beg, beg + c);
    }
    wave_sync();
}

// a share's first output slot
__device__ __forceinline__ u32 share_base(const PassBufs &b, u32 tile, int wv)
{
    u64 base = b.t_base[tile / STS_BKT_CHUNK] + b.t_off[tile];
    for (int w = 0; w < wv; ++w) base += b.w_kept[(tile << 2) + (u32)w];
    return (u32)base;
}

// when the window held the cut, the survivors are in the wave's slab: all
// entries above the window, and the window's by the threshold; or every candidate
// is there, as the window's
template <typename AT>
__device__ __forceinline__ void copy_share(const BktPlan &p, const PassBufs &b, u32 tile, int wv, u32 *cnt, u64 thr_w,
                                           u64 thr_k, bool rescale, double scale)
{
    constexpr int UN = 8; // items of a share held in registers, per lane
    const u32 lane = (u32)sts_lane();
    const int bits = 2 + p.delta, shift = b.slab_shift;
    const u32 sl = (tile << 2) + (u32)wv;
    cnt[lane] = 0;
    const u32 na = uni(b.t_above[sl]), ns = uni(b.t_side[sl]), n = na + ns;
    if (n == 0) { // empty buckets may begin anywhere
        if (lane < 4u << p.delta) {
            const u32 in = bkt_rep(p, tile) ^ bkt_comb(p, (lane & 3u) | ((u32)wv << 2));
            b.bd_out[(in << p.delta) | (lane >> 2)] = make_uint2(0, 0);
        }
        return;
    }
    const u32 base = uni(share_base(b, tile, wv));
    wave_sync();
    const u32 cap = (u32)b.out_cap;
    u64 *ok = b.out_keys;
    AT *oa = (AT *)b.out_amps;
    const u64 slab = (u64)sl << shift;
    const u64 *sk = b.side_key + slab, *sw = b.side_w + slab;
    const AT *sa = (const AT *)b.side_amp + slab;
    const u32 ab0 = (1u << shift) - na; // the entries above the window
    auto place = [&](u32 j) { return j < na ? ab0 + j : j - na; };
    if (n <= UN * 64) {
        u64 kk[UN], ww[UN];
        AT aa[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            const u32 j = (u32)r * 64 + lane;
            ww[r] = ~0ull; // above the window: kept
            if (j < n) {
                const u32 i = place(j);
                kk[r] = __builtin_nontemporal_load(&sk[i]);
                aa[r].x = __builtin_nontemporal_load(&sa[i].x);
                aa[r].y = __builtin_nontemporal_load(&sa[i].y);
                if (j >= na) ww[r] = __builtin_nontemporal_load(&sw[i]);
            }
        }
        u32 pos[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            pos[r] = ~0u;
            if ((u32)r * 64 < n) { // uniform
                const bool keep = (u32)r * 64 + lane < n && survives<AT>(ww[r], kk[r], false, thr_w, thr_k);
                const u32 sub = keep ? sub_bucket(p, kk[r]) : 0u;
                const u32 rank = sub_rank(keep, sub, bits, cnt);
                if (keep) pos[r] = rank | (sub << 26); // ranks are below UN * 64
            }
        }
        wave_sync();
        sub_starts(p, b, tile, wv, base, cnt);
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            if (pos[r] == ~0u) continue;
            const u32 at = cnt[pos[r] >> 26] + (pos[r] & ((1u << 26) - 1u));
            if (at < cap) {
                ok[at] = kk[r];
                const AT o = out_amp(aa[r], rescale, scale);
                oa[at] = o;
            }
        }
        return;
    }
    // a large share: count, then place
    for (int phase = 0; phase < 2; ++phase) {
        for (u32 j0 = 0; j0 < n; j0 += UN * 64) {
            u64 kk[UN], ww[UN];
            AT aa[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = j0 + (u32)r * 64 + lane;
                ww[r] = ~0ull;
                if (j < n) {
                    const u32 i = place(j);
                    kk[r] = sk[i];
                    if (j >= na) ww[r] = sw[i];
                    if (phase) aa[r] = sa[i];
                }
            }
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = j0 + (u32)r * 64 + lane;
                if (j0 + (u32)r * 64 >= n) break; // uniform
                const bool keep = j < n && survives<AT>(ww[r], kk[r], false, thr_w, thr_k);
                const u32 at = sub_rank(keep, keep ? sub_bucket(p, kk[r]) : 0u, bits, cnt);
                if (phase && keep && at < cap) {
                    ok[at] = kk[r];
                    oa[at] = out_amp(aa[r], rescale, scale);
                }
            }
        }
        wave_sync();
        if (phase == 0) sub_starts(p, b, tile, wv, base, cnt);
    }
}

// whether the survivors are in the slabs
__device__ __forceinline__ bool in_slabs(const PassBufs &b, const DevCtl *ctl)
{
    const int keep_all = ctl->keep_all, hit = ctl->pred_hit, every = ctl->slab_all;
    return b.materialise || keep_all ? every : hit || every;
}

// Bound by memory: 536 MB in 120 us (4.5 TB/s) at 2^24 complex64 terms. The
// slabs are read past the caches, the survivors are not written past them: with
// non-temporal amplitude stores the copy took 143 us and the next weighing pass 323
// instead of 330.
template <typename AT>
__global__ void __launch_bounds__(STS_WG) k_bkt_copy(const GateArg *__restrict__ gp, PassBufs b)
{
    __shared__ u32 s_cnt[BW][BW_SUBS];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const DevCtl *ctl = b.ctl;
    const bool all = b.materialise || ctl->keep_all;
    if (!in_slabs(b, ctl)) return; // uniform
    copy_share<AT>(gp->bkt, b, blockIdx.x, wv, s_cnt[wv], all ? 0ull : ctl->thr_wbits, all ? ~0ull : ctl->thr_key,
                   !all && ctl->dropped, ctl->scale);
}

// otherwise they are computed again
template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_emit(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    const BktPlan &p = g.bkt;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, BW> s;
    __shared__ u32 s_cnt[BW][BW_SUBS];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const DevCtl *ctl = b.ctl;
    const int keep_all = ctl->keep_all, dropped = ctl->dropped;
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const double scale = ctl->scale;
    const bool all = b.materialise || keep_all;
    const bool rescale = !all && dropped;
    const u32 cap = (u32)b.out_cap, ntiles = bkt_tiles(p);
    if (in_slabs(b, ctl)) { // uniform: the copy's part (of a small step; else k_bkt_copy does it)
        if (b.emit_copies)
            for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
                copy_share<AT>(p, b, tile, wv, s_cnt[wv], thr_w, thr_k, rescale, scale);
        return;
    }
    smem_begin<AT, M, BW>(s, g);
    __syncthreads();
    const int bits = 2 + p.delta;
    u64 *ok = b.out_keys;
    AT *oa = (AT *)b.out_amps;
    u32 *cnt = s_cnt[wv];
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        cnt[sts_lane()] = 0;
        const u32 base = uni(share_base(b, tile, wv));
        wave_sync();
        const Share sh = load_share(p, b.bd_in, tile, wv);
#pragma unroll 1
        for (int phase = 0; phase < 2; ++phase) {
            share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, b.keys, (const AT *)b.amps,
                                [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
                for (int i = 0; i < (1 << M); ++i) {
                    AT o;
                    o.x = ox[i];
                    o.y = oy[i];
                    const u64 key = rest | pattern_bits<M>(gl, i);
                    const bool keep =
                        active && nonzero(o) && survives<AT>(weight_bits(o), key, all, thr_w, thr_k);
                    const u32 at = sub_rank(keep, keep ? sub_bucket(p, key) : 0u, bits, cnt);
                    if (phase && keep && at < cap) {
                        ok[at] = key;
                        oa[at] = out_amp(o, rescale, scale);
                    }
                }
            });
            wave_sync();
            if (phase == 0) sub_starts(p, b, tile, wv, base, cnt);
        }
    }
}

// ---------------------------------------------------------------------------
// Small steps (at most STS_SEL_SHARES shares). The weighing pass bins the
// weights as the histogram pass does and copies a window of weights and the
// candidates above it to the slabs: two octaves around the previous cut
// (k_bkt_small; everything without a previous cut), or, of larger states, the
// bin that the sampling pass, run on all terms, found (k_bkt_mid, which also
// sums the mass above it). One workgroup then does the whole selection: the
// level-1 pick over the exponent bins, the further levels over the window's
// entries of the cut's exponent, and the survivors' offsets. Several short
// launches in a chain cost more than one workgroup's passes over some thousands
// of entries. (Selecting in the weighing pass's last workgroup instead of a
// launch of its own was slower: 48 us instead of 12 + 29 at 4096 terms; the
// fences of that handover cost more than the launch.) A window that missed the
// cut is not recovered by further launches either: the selection then computes
// the candidates again and fills the slabs with those of the cut's exponent and
// above (for every pass over them if a slab cannot hold its share's).
//
// The selection is bound by what its waves issue on one CU and by round trips
// to memory, so its first loads go out together, entries are kept on the chip
// (a two-octave window's in registers, a found one's in an LDS list), and 512
// threads do the work: 31 us at 16,384 terms, 43 with 1024 threads that read the
// entries again for each pass; 33 us at 100,003 terms, where the chain of
// launches it replaced took 55. A miss: 200 us at 16,384 terms, 620 when the
// candidates were computed again for each pass.
// ---------------------------------------------------------------------------
constexpr int SEL_NT = 512;
constexpr int SEL_S = 32; // shares of which a wave holds up to 64 entries each

constexpr int SEL_NW = SEL_NT / 64;
constexpr u32 SEL_LIST = 8192; // entries of a sampled window that LDS holds
constexpr int MID_GROUPS = 512; // most workgroups of k_bkt_mid
__host__ __device__ __forceinline__ int mid_groups(u32 tiles) { return tiles < MID_GROUPS ? (int)tiles : MID_GROUPS; }


template <typename AT> struct SelectSmem {
    union {
        sts_select::Level1Smem<SEL_NT> l1;
        BktSmem<AT, SEL_NW> bkt; // when candidates are computed again
        struct {
            u64 w[SEL_LIST];
            unsigned short at[SEL_LIST]; // share << 5 | index in its slab
        } list; // a sampled window's entries
    } u;
    __attribute__((aligned(16))) unsigned char raw[sts_select::THIN_BINS * 12];
    sts_select::Level1Cut l1;
    sts_select::CutSmem cut;
    sts_select::Sub sub;
    __attribute__((aligned(16))) u128 last[STS_FINAL_SORT]; // the terms the cut is among,
    u32 last_share[STS_FINAL_SORT];                         // and their shares
    u32 kept[STS_SEL_SHARES];
    u32 side[STS_SEL_SHARES]; // window entries of each share's slab
    u32 first[STS_SEL_SHARES]; // its first entry in the list
    u32 full;                 // a slab could not hold them
    u64 scan[SEL_NW];
};

template <typename AT, int M, bool MID>
__global__ void __launch_bounds__(SEL_NT) k_bkt_select(const GateArg *__restrict__ gp, PassBufs b)
{
    using namespace sts_select;
    constexpr int NT = SEL_NT, S = SEL_S;
    static_assert(STS_SEL_SHARES <= 1 << 11, "a share and an index below 32 in 16 bits");
    const GateArg &g = *gp;
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ SelectSmem<AT> m;
    BktSmem<AT, SEL_NW> &s = m.u.bkt;
    DevCtl *ctl = b.ctl;
    const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const u32 lane = (u32)sts_lane();
    const u32 ntiles = bkt_tiles(g.bkt), nsl = ntiles << 2;
    const int shift = b.slab_shift;
    // control words, read before the pick writes any
    const int e_prev = ctl->e_pred, e_w = small_window(ctl);
    const bool sampled = MID && ctl->w_mode;
    const u32 over = ctl->w_over;
    const u64 K = ctl->K;
    const double l10 = ctl->log10_cum;
    // Every load the selection starts with is issued at once: the exponent
    // bins, the shares' counts, and the first 64 window entries of S shares
    // per wave, which stay in registers for all passes over the entries (a
    // sampled window's are few, and scattered: read again by each pass)
    const EarlyBins<NT> bins(b.h1);
    const u32 room = 1u << shift;
    const u32 sl_own = lane * (NT / 64) + (u32)wv; // the share whose count the lane holds
    u32 ns0 = lane < (u32)S && sl_own < nsl ? b.t_side[sl_own] : 0u;
    u64 wa[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
        const u32 sl = (u32)(i * (NT / 64) + wv);
        wa[i] = !MID && sl < nsl && lane < room ? b.side_w[((u64)sl << shift) + lane] : ~0ull;
    }
    for (u32 sl = t; sl < nsl; sl += NT) {
        m.side[sl] = std::min(b.t_side[sl], room);
        m.kept[sl] = b.t_above[sl];
    }
    for (int i = t; i < THIN_BINS * 3 / 2; i += NT) reinterpret_cast<u64 *>(m.raw)[i] = 0;
    ns0 = std::min(ns0, room);
    pick_level1<NT>(b, sampled ? mid_groups(ntiles) : 0, 0, sampled ? 2 : 0, m.u.l1, bins);
#pragma unroll
    for (int i = 0; i < S; ++i) { // no weight has all bits set
        if (lane >= sts_readlane(ns0, i)) wa[i] = ~0ull;
    }
    __syncthreads();
    if (t < (int)(sizeof(Level1Cut) / sizeof(u64)))
        reinterpret_cast<u64 *>(&m.l1)[t] = reinterpret_cast<const u64 *>(&m.u.l1.cut)[t];
    if (t == 0) m.full = over;
    __syncthreads();
    const bool all = m.l1.keep_all;
    const int e = m.l1.e;
    auto recompute = [&](auto begin, auto body, auto end) __attribute__((always_inline)) { // of every share and candidate
        for (u32 sl = (u32)wv; sl < nsl; sl += SEL_NW) {
            const Share sh = load_share(g.bkt, b.bd_in, sl >> 2, (int)(sl & 3u));
            begin(sl);
            share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, b.keys, (const AT *)b.amps,
                                [&](const auto &ox, const auto &oy, u64 rest, bool active) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < (1 << M); ++i) {
                    AT o;
                    o.x = ox[i];
                    o.y = oy[i];
                    body(sl, weight_bits(o), rest | pattern_bits<M>(gl, i), o, active && nonzero(o));
                }
            });
            end(sl);
        }
    };
    // whether the slabs hold every candidate of the cut's exponent and above;
    // when the window missed, they are filled again with those
    const bool hit = all || (MID ? !sampled || m.l1.in_window : e_prev < 0 || e == e_w || e == e_w + 1);
    const bool win = MID && sampled && hit && !over; // the cut lies in the sampled window
    // such a window has a few entries a share: they are listed in LDS, four
    // lanes a share, so that the passes over them run without gaps
    u32 listed = 0;
    if (win && !all) {
        constexpr u32 PER = STS_SEL_SHARES / NT; // neighbouring shares of a thread
        u32 ns[PER], sum = 0, most = 0;
#pragma unroll
        for (u32 r = 0; r < PER; ++r) {
            const u32 sl = (u32)t * PER + r;
            ns[r] = sl < nsl ? m.side[sl] : 0u;
            sum += ns[r];
            most = std::max(most, ns[r]);
        }
        if (t == 0) m.full = 0;
        __syncthreads(); // (the bins' lists are read: the list takes their place)
        if (most >= 32) m.full = 1;
        u32 total, first = block_excl_scan<u32, NT>(sum, reinterpret_cast<u32 *>(m.scan), &total);
#pragma unroll
        for (u32 r = 0; r < PER; ++r) {
            m.first[(u32)t * PER + r] = first;
            first += ns[r];
        }
        __syncthreads();
        listed = total <= SEL_LIST && !m.full ? total : 0u;
        if (listed) {
            constexpr u32 LN = 4, ROUNDS = STS_SEL_SHARES / (NT / LN);
            const u32 own = (u32)t / LN, l = (u32)t % LN;
            u64 w[ROUNDS];
#pragma unroll
            for (u32 r = 0; r < ROUNDS; ++r) { // every share's load in flight at once
                const u32 sl = own + r * (NT / LN);
                w[r] = sl < nsl && l < room ? b.side_w[((u64)sl << shift) + l] : 0ull;
            }
#pragma unroll
            for (u32 r = 0; r < ROUNDS; ++r) {
                const u32 sl = own + r * (NT / LN);
                const u32 n = sl < nsl ? m.side[sl] : 0u;
                for (u32 i = l; i < n; i += LN) {
                    const u32 at = m.first[sl] + i;
                    m.u.list.w[at] = i < LN ? w[r] : b.side_w[((u64)sl << shift) + i];
                    m.u.list.at[at] = (unsigned short)(sl << 5 | i);
                }
            }
        }
        __syncthreads();
        if (t == 0) m.full = 0;
        __syncthreads();
    }

    if (!hit || over) { // uniform
        smem_begin<AT, M, SEL_NW>(s, g);
        __syncthreads();
    }
    if (!hit && !over) {
        SlabOut so;
        recompute([&](u32) __attribute__((always_inline)) { so = SlabOut{0, 0, 0, true}; },
                  [&](u32 sl, u64 w, u64 k, const AT &o, bool valid) __attribute__((always_inline)) {
                      const int x = (int)(w >> 52);
                      const u64 at = (u64)sl << shift;
                      slab_put<AT>(so, b.side_key + at, b.side_w + at, (AT *)b.side_amp + at, room, valid && x == e,
                                   valid && x > e, k, w, o);
                  },
                  [&](u32 sl) __attribute__((always_inline)) {
                      if (lane == 0) {
                          b.t_above[sl] = m.kept[sl] = so.c_ab;
                          b.t_side[sl] = so.c_in;
                          m.side[sl] = std::min(so.c_in, room);
                          if (!so.fits) m.full = 1;
                      }
                  });
        __threadfence_block();
        __syncthreads();
    }
    const bool slabs = !all && !m.full;
    // block(first share, first index, counts, w[S]) for 64 window entries of S
    // shares (NT / 64 apart) at a time: those held in registers, then others.
    // counts: lane i's is the i-th share's, entries past it have all bits set.
    auto entries = [&](auto block) __attribute__((always_inline)) {
        for (u32 sl0 = (u32)wv; sl0 < nsl; sl0 += (u32)(S * (NT / 64))) {
            const u32 sl = sl0 + lane * (NT / 64);
            const u32 ns = lane < (u32)S && sl < nsl ? m.side[sl] : 0u;
            for (u32 c0 = 0; wballot(ns > c0); c0 += 64) {
                u64 w[S];
                const u32 at = c0 + lane;
                if (!MID && c0 == 0 && sl0 == (u32)wv && hit) {
#pragma unroll
                    for (int i = 0; i < S; ++i) w[i] = wa[i];
                } else {
#pragma unroll
                    for (int i = 0; i < S; ++i)
                        w[i] = at < sts_readlane(ns, i)
                                   ? b.side_w[((u64)(sl0 + (u32)(i * (NT / 64))) << shift) + at] : ~0ull;
                }
                block(sl0, c0, ns, w);
            }
        }
    };
    if (!all) {
        if (t == 0) {
            m.sub.cnt_before = win ? m.l1.w_cnt : m.l1.cnt;
            m.sub.mb = win ? make128(m.l1.w_mb_lo, m.l1.w_mb_hi) : (u128)0;
            m.sub.vpre = 0;
            m.sub.vshift = 116;
            m.sub.count = win ? m.l1.w_count : m.l1.count;
        }
        __syncthreads();
        // the weights of the subset under a prefix: from lo up to below hi (where
        // the key decides, of those with the prefix's weight)
        auto bounds = [&](int vshift, u128 vpre, u64 &lo, u64 &hi) __attribute__((always_inline)) {
            const int sh = vshift < 64 ? 0 : vshift - 64;
            const u64 top = (u64)(vshift < 64 ? vpre >> (64 - vshift) : vpre);
            lo = ((u64)e << 52) | ((((1ull << (52 - sh)) - 1) - top) << sh);
            hi = lo + (1ull << sh);
        };
        auto place = [&](u32 i) __attribute__((always_inline)) { // of a listed entry in the side buffer
            const u32 at = m.u.list.at[i];
            return ((u64)(at >> 5) << shift) + (at & 31u);
        };
        auto each = [&](int vshift, u128 vpre, bool keyed, auto f) __attribute__((always_inline)) {
            if (!slabs) {
                recompute([](u32) {},
                          [&](u32, u64 w, u64 k, const AT &, bool valid) __attribute__((always_inline)) {
                              const u128 v = rank_key(w, k);
                              if (valid && (int)(w >> 52) == e && (v >> vshift) == vpre) f(v);
                          },
                          [](u32) {});
                return;
            }
            u64 lo, hi;
            bounds(vshift, vpre, lo, hi);
            if (listed) {
                for (u32 i = t; i < listed; i += NT) {
                    const u64 w = m.u.list.w[i];
                    if (w - lo >= hi - lo) continue;
                    const u64 k = keyed ? b.side_key[place(i)] : 0ull;
                    const u128 v = rank_key(w, k);
                    if (vshift >= 64 || (v >> vshift) == vpre) f(v);
                }
                return;
            }
            if (vshift == 116) {
                entries([&](u32, u32 c0, u32 ns, const u64 (&w)[S]) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < S; ++i)
                        if (sts_readlane(ns, i) > c0 && (u32)(w[i] >> 52) == (u32)e) f.first(w[i]);
                });
                return;
            }
            entries([&](u32 sl0, u32 i0, u32, const u64 (&w)[S]) __attribute__((always_inline)) {
                u32 in = 0;
#pragma unroll
                for (int i = 0; i < S; ++i) in |= w[i] - lo < hi - lo ? 1u << i : 0u;
                while (in) { // a few: the first level took most
                    const u32 i = (u32)__builtin_ctz(in);
                    const u64 at = ((u64)(sl0 + i * (NT / 64)) << shift) + i0 + lane;
                    in &= in - 1;
                    const u128 v = rank_key(b.side_w[at], keyed ? b.side_key[at] : 0ull);
                    if (vshift >= 64 || (v >> vshift) == vpre) f(v);
                }
            });
        };
        const u128 R = make128(m.l1.R_lo, m.l1.R_hi);
        bool ok = narrow_cut<NT, true>(each, e, K, R, m.sub, m.raw, m.cut, STS_FINAL_SORT, true);
        const int vshift = m.sub.vshift;
        const u128 vpre = m.sub.vpre;
        const u32 count = (u32)m.sub.count;
        if (t == 0) {
            m.cut.n = 0;
            m.cut.hit = 0xffffffffu;
        }
        __syncthreads();
        if (ok && count <= STS_FINAL_SORT) {
            // list the subset and, in the same pass, count the survivors
            // ranked before it, share by share
            auto sort_out = [&](u32 sl, u64 w, u64 k, u32 &before) __attribute__((always_inline)) {
                const int x = (int)(w >> 52);
                const u128 p = rank_key(w, k) >> vshift;
                if (x > e || (x == e && p < vpre)) {
                    ++before;
                } else if (x == e && p == vpre) {
                    const u32 slot = atomicAdd(&m.cut.n, 1u);
                    if (slot < STS_FINAL_SORT) {
                        m.last[slot] = rank_key(w, k);
                        m.last_share[slot] = sl;
                    }
                }
            };
            if (slabs) {
                // by the weight's high word; what that leaves open (the subset,
                // as a rule) by all of it
                u64 lo, hi;
                bounds(vshift, vpre, lo, hi);
                const u32 lo32 = (u32)(lo >> 32), top32 = (u32)((hi - 1) >> 32);
                if (listed) {
                    for (u32 i = t; i < listed; i += NT) {
                        const u64 w = m.u.list.w[i];
                        if (w < lo) continue;
                        const u32 sl = (u32)m.u.list.at[i] >> 5;
                        u32 before = w >= hi ? 1u : 0u;
                        if (!before) sort_out(sl, w, b.side_key[place(i)], before);
                        if (before) atomicAdd(&m.kept[sl], 1u);
                    }
                } else entries([&](u32 sl0, u32 i0, u32 ns, const u64 (&w)[S]) __attribute__((always_inline)) {
                    u32 above = 0; // of lane i: the i-th share's
                    u32 near = 0;
#pragma unroll
                    for (int i = 0; i < S; ++i) {
                        if (sts_readlane(ns, i) <= i0) continue;
                        const u32 h = (u32)(w[i] >> 32);
                        near |= h - lo32 <= top32 - lo32 ? 1u << i : 0u;
                        const u32 n = (u32)__popcll(wballot((int)h > (int)top32));
                        above = lane == (u32)i ? n : above;
                    }
                    if (lane < (u32)S && above) atomicAdd(&m.kept[sl0 + lane * (NT / 64)], above);
                    while (near) {
                        const u32 i = (u32)__builtin_ctz(near);
                        near &= near - 1;
                        const u32 sl = sl0 + i * (NT / 64);
                        const u64 at = ((u64)sl << shift) + i0 + lane;
                        u32 before = 0;
                        sort_out(sl, b.side_w[at], b.side_key[at], before);
                        if (before) atomicAdd(&m.kept[sl], 1u);
                    }
                });
            } else {
                for (u32 sl = t; sl < nsl; sl += NT) m.kept[sl] = 0;
                __syncthreads();
                recompute([](u32) {},
                          [&](u32 sl, u64 w, u64 k, const AT &, bool valid) __attribute__((always_inline)) {
                              u32 before = 0;
                              if (valid) sort_out(sl, w, k, before);
                              const u64 mk = wballot(before != 0);
                              if (lane == 0) m.kept[sl] += (u32)__popcll(mk); // the share is this wave's
                          },
                          [](u32) {});
            }
            __syncthreads();
            ok = m.cut.n == count;
            const u32 rank = rank_cut<NT>(m.last, count, e, K, R, m.sub, m.cut);
            ok = ok && m.cut.hit != 0xffffffffu;
            if (ok && rank <= m.cut.hit) atomicAdd(&m.kept[m.last_share[t]], 1u);
        } else {
            ok = false; // no subset is larger once every bit of V is fixed
        }
        if (!ok) { // uniform; an internal inconsistency: reported, and no term kept
            for (u32 sl = t; sl < nsl; sl += NT) m.kept[sl] = 0;
            if (t == 0) {
                atomicOr(&ctl->flags, STS_F_UNRESOLVED);
                ctl->thr_wbits = ~0ull;
                ctl->thr_key = 0;
            }
        }
        if (ok && wv == NT / 64 - 1) finish_cut(ctl, m.cut, e, m.l1.S, m.l1.total, m.l1.W, l10);
    } else {
        for (u32 sl = t; sl < nsl; sl += NT) m.kept[sl] = b.w_all[sl];
    }
    __syncthreads();
    // offsets: one tile per thread
    u64 carry = 0;
    for (u32 t0 = 0; t0 < ntiles; t0 += NT) {
        const u32 tile = t0 + (u32)t;
        u32 k[4] = {0, 0, 0, 0};
        if (tile < ntiles) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                k[w] = m.kept[(tile << 2) + w];
                b.w_kept[(tile << 2) + w] = k[w];
            }
        }
        const u64 sum = (u64)k[0] + k[1] + k[2] + k[3];
        u64 total;
        const u64 at = block_excl_scan<u64, NT>(sum, m.scan, &total) + carry;
        if (tile < ntiles) b.t_off[tile] = at;
        if (tile < ntiles && tile % STS_BKT_CHUNK == 0) b.t_base[tile / STS_BKT_CHUNK] = 0;
        carry += total;
    }
    if (t == 0) {
        *b.n_out = carry;
        if (carry > b.out_cap && !b.may_refuse) atomicOr(&ctl->flags, STS_F_OUT_OVERFLOW);
        ctl->w_over = 0;
        ctl->slab_all = 0;
        ctl->pred_hit = slabs;
    }
}

template <typename AT, int M, bool MID>
__device__ __forceinline__ void small_pass(const GateArg &g, const PassBufs &b)
{
    const GateLoc<M> gl = gate_loc<M>(g);
    __shared__ BktSmem<AT, BW> s;
    __shared__ u64 s_hi[TT_SLOTS], s_lo[TT_SLOTS];
    __shared__ u64 s_win[9]; // as pick_level1 takes them
    DevCtl *ctl = b.ctl;
    smem_begin<AT, M, BW>(s, g);
    for (int i = threadIdx.x; i < TT_SLOTS; i += STS_WG) {
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
    const u64 *keys = b.keys;
    const AT *amps = (const AT *)b.amps;
    const u32 nsl = bkt_tiles(g.bkt) << 2;
    const int e_prev = ctl->e_pred;
    const int e_w = small_window(ctl);
    // the window, in the weight's high word (whose bits decide it); without a
    // previous cut or a sample's window, everything
    const bool sampled = MID && ctl->w_mode;
    u32 wL = 0u, wH = ~0u;
    if (sampled) {
        wL = (u32)(ctl->w_lo >> 32);
        wH = (u32)(ctl->w_hi >> 32) + 1u;
    } else if (!MID && e_prev >= 0) {
        wL = (u32)e_w << 20;
        wH = (u32)(e_w + 2) << 20;
    }
    wL = uni(wL);
    wH = uni(wH);
    // the sampled window's (upper) exponent, and mantissa sums in it above the
    // window and inside, and inside in the exponent below
    const u32 e_beg = uni(((wH - 1u) >> 20) << 20), e_end = e_beg + (1u << 20);
    u64 ab_hi = 0, ab_lo = 0, in_hi = 0, in_lo = 0, un_hi = 0, un_lo = 0;
    u32 n_ab = 0, n_in = 0, n_un = 0;
    if (threadIdx.x < 9) s_win[threadIdx.x] = 0;
    const int shift = b.slab_shift;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int hot_lo = (e_prev >= 0 ? e_prev : TT_EBASE + 116) - (TT_HOT - 4);
    __syncthreads();
    // (a wave's shares go to the LDS bins while those stay exact: the grid
    // gives it a few)
    for (u32 sl = blockIdx.x * BW + (u32)wv; sl < nsl; sl += gridDim.x * BW) {
        const Share sh = load_share(g.bkt, b.bd_in, sl >> 2, (int)(sl & 3u));
        const u64 slab = (u64)sl << shift;
        const bool direct = sh.n > BW_BINNED;
        u64 *const sk = b.side_key + slab;
        u64 *const sw = b.side_w + slab;
        AT *const sa = (AT *)b.side_amp + slab;
        SlabOut so = {0, 0, 0, true};
        share_groups<AT, M>(s.w[wv], s.ucol, gl, sh, keys, amps,
                            [&](const auto &ox, const auto &oy, u64 rest, bool active) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                AT o;
                o.x = ox[i];
                o.y = oy[i];
                const bool cand = active && nonzero(o);
                const u64 wb = weight_bits(o);
                const u32 hw = (u32)(wb >> 32);
                if (cand) bin_weight(b, s_hi, s_lo, hot_lo, wb, direct);
                so.c_all += (u32)__popcll(wballot(cand));
                if (sampled && cand && hw >= wL && hw < e_end) { // uniform, then of some lanes
                    const u64 mant = sts_mant(wb);
                    const bool un = hw < e_beg, in = hw < wH && !un, ab = hw >= wH;
                    const u64 h = mant >> 26, l = mant & ((1ull << 26) - 1);
                    in_hi += in ? h : 0ull;
                    in_lo += in ? l : 0ull;
                    ab_hi += ab ? h : 0ull;
                    ab_lo += ab ? l : 0ull;
                    if (un) { // (seldom of any lane)
                        un_hi += h;
                        un_lo += l;
                        ++n_un;
                    }
                }
                slab_put<AT>(so, sk, sw, sa, 1u << shift, cand && hw >= wL && hw < wH, cand && hw >= wH,
                             rest | pattern_bits<M>(gl, i), wb, o);
            }
        });
        if (sts_lane() == 0) {
            b.w_all[sl] = so.c_all;
            b.t_above[sl] = so.c_ab;
            b.t_side[sl] = so.c_in;
            n_ab += so.c_ab;
            n_in += so.c_in;
            if (!so.fits) atomicOr(&ctl->w_over, 1u);
        }
    }
    if (sampled) {
        const bool l0 = sts_lane() == 0; // (the counts are the wave's)
        u64 v[9] = {l0 ? n_ab : 0u, ab_hi, ab_lo, (l0 ? n_in : 0u) - (u64)n_un, in_hi, in_lo, n_un, un_hi, un_lo};
#pragma unroll
        for (int f = 0; f < 9; ++f) {
            v[f] = wave_incl_scan(v[f]);
            if (sts_lane() == 63) atomicAdd((unsigned long long *)&s_win[f], (unsigned long long)v[f]);
        }
    }
    __syncthreads();
    if (sampled && threadIdx.x < 9) b.wpart[threadIdx.x * STS_MAX_GROUPS + blockIdx.x] = s_win[threadIdx.x];
    flush_bins(b, s_hi, s_lo, hot_lo);
}

// Both are as long as one share's chain of LDS round trips and the flush of the
// bins: 11 us at 4,096 to 16,384 terms, k_bkt_mid 18 at 100,003 (k_bkt_weigh, whose
// tables fill a CU's LDS, took 27 there).
template <typename AT, int M> __global__ void __launch_bounds__(STS_WG) k_bkt_small(GateArg g, PassBufs b)
{
    if (blockIdx.x == 0) put_gate(g, b.gate_dst);
    small_pass<AT, M, false>(g, b);
}

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_mid(const GateArg *__restrict__ gp, PassBufs b)
{
    small_pass<AT, M, true>(*gp, b);
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
// workgroups of a persistent pass that are resident at once
template <typename F> int resident_groups(F kernel, int threads)
{
    int per_cu = 0, dev = 0, cus = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0);
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return std::min((per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1), STS_MAX_GROUPS);
}

// of the histogram, extraction, counting and emission passes
template <typename AT, int M> int pass_capacity(int kind)
{
    static const int hist = resident_groups(k_bkt_hist<AT, M>, STS_WG);
    static const int extract = resident_groups(k_bkt_extract<AT, M>, STS_WG);
    static const int count = resident_groups(k_bkt_count<AT, M>, STS_WG);
    static const int emit = resident_groups(k_bkt_emit<AT, M>, STS_WG);
    return kind == STS_BKT_HIST ? hist : kind == STS_BKT_EXTRACT ? extract : kind == STS_BKT_COUNT ? count : emit;
}

template <typename AT, int M> int weigh_capacity()
{
    static const int cap = resident_groups(k_bkt_weigh<AT, M>, 64 * WeighWaves<AT>::value);
    return cap;
}

template <typename AT, int M> int weigh_grid(int tiles)
{
    constexpr int per = WeighWaves<AT>::value / 4;
    return std::min((tiles + per - 1) / per, weigh_capacity<AT, M>());
}

template <typename AT, int M> const void *first_kernel(int kind)
{
    return kind == STS_BKT_SAMPLE ? reinterpret_cast<const void *>(&k_bkt_sample<AT, M>)
                                  : reinterpret_cast<const void *>(&k_bkt_small<AT, M>);
}

template <typename AT, int M>
hipError_t launch_m(int kind, const PassBufs &b, int tiles, hipStream_t s, const GateArg *first)
{
    // a pass over tiles by all the workgroups that are resident at once, also
    // where it is launched in case a window missed (exiting at once takes as long
    // in one workgroup per CU, and a miss at 2^24 terms took 4.4 instead of 2.4 ms
    // when each of them computed the candidates again; now it adds 1.0 ms)
    const int cap = pass_capacity<AT, M>(kind);
    // the sample's tiles: at 2^24 terms twice as many halve the misses for 1 us
    // of 550, at 2^20 they cost as much as they save
    const int sample = b.fine_window ? tiles : tiles >= 1 << 14 ? STS_SAMPLE_TILES : STS_SAMPLE_TILES / 2;
    switch (kind) {
    case STS_BKT_HIST:
        hipLaunchKernelGGL((k_bkt_hist<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_SAMPLE:
        hipLaunchKernelGGL((k_bkt_sample<AT, M>), dim3(sample), dim3(STS_WG), 0, s, *first, b);
        break;
    case STS_BKT_EXTRACT:
        hipLaunchKernelGGL((k_bkt_extract<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_COUNT:
        hipLaunchKernelGGL((k_bkt_count<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_WEIGH:
        hipLaunchKernelGGL((k_bkt_weigh<AT, M>), dim3(weigh_grid<AT, M>(tiles)),
                           dim3(64 * WeighWaves<AT>::value), 0, s,
                           b.gate, b);
        break;
    case STS_BKT_COPY:
        hipLaunchKernelGGL((k_bkt_copy<AT>), dim3(tiles), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_SMALL:
        hipLaunchKernelGGL((k_bkt_small<AT, M>), dim3(std::min(tiles, 256)), dim3(STS_WG), 0, s, *first, b);
        break;
    case STS_BKT_SELECT:
        hipLaunchKernelGGL((k_bkt_select<AT, M, false>), dim3(1), dim3(SEL_NT), 0, s, b.gate, b);
        break;
    case STS_BKT_MID:
        hipLaunchKernelGGL((k_bkt_mid<AT, M>), dim3(mid_groups((u32)tiles)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_SELECT_MID:
        hipLaunchKernelGGL((k_bkt_select<AT, M, true>), dim3(1), dim3(SEL_NT), 0, s, b.gate, b);
        break;
    case STS_BKT_EMIT:
        hipLaunchKernelGGL((k_bkt_emit<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

} // namespace sts_bucket
