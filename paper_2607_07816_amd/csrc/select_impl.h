// select_impl.h - parts of the cut's selection shared by its kernels: exact
// masses held by a wave, digit picks, the level-1 pick, and the last levels.
#pragma once
#include "kernels.h"

namespace sts_select {

// bit position of the unit 2^(max(e,1)-1075) on the 2^-1074 grid
__device__ __forceinline__ int unit_bit(int e) { return (e > 0 ? e : 1) - 1; }

__device__ __forceinline__ u128 make128(u64 lo, u64 hi) { return ((u128)hi << 64) | lo; }

// ---------------------------------------------------------------------------
// Exact masses, one wave wide: a number of 64 limbs of 64 bits (units
// 2^-1074), limb i held by lane i. Every lane of the wave takes part in each
// operation. Carries between limbs are resolved at once from two ballots: a
// limb generates a carry (its sum wrapped) or propagates one (its sum is all
// ones), and the carries into the limbs are the carries of the binary sum
// (G | P) + G, i.e. ((G | P) + G) ^ (G | P) ^ G.
// ---------------------------------------------------------------------------
__device__ __forceinline__ u64 wl_carry_in(bool gen, bool prop)
{
    const u64 G = __ballot(gen), P = __ballot(prop);
    const u64 X = G | P;
    return (((X + G) ^ X ^ G) >> sts_lane()) & 1ull;
}

__device__ __forceinline__ u64 wl_add(u64 a, u64 b)
{
    const u64 s = a + b;
    return s + wl_carry_in(s < a, s == ~0ull);
}

// a - b, a >= b
__device__ __forceinline__ u64 wl_sub(u64 a, u64 b)
{
    const u64 d = a - b;
    return d - wl_carry_in(a < b, d == 0);
}

// this lane's limb of v * 2^bit, v < 2^128 given as (lo, hi)
__device__ __forceinline__ u64 wl_piece(u64 lo, u64 hi, int bit)
{
    const int k = sts_lane() - (bit >> 6), off = bit & 63;
    if (k == 0) return lo << off;
    if (k == 1) return off ? (hi << off) | (lo >> (64 - off)) : hi;
    if (k == 2) return off ? hi >> (64 - off) : 0ull;
    return 0ull;
}

// sign of a - b
__device__ __forceinline__ int wl_cmp(u64 a, u64 b)
{
    const u64 D = __ballot(a != b);
    if (!D) return 0;
    const int top = 63 - __clzll((long long)D);
    return ((__ballot(a > b) >> top) & 1ull) ? 1 : -1;
}

// limb `src` of the number (0 outside 0..63); src may differ between lanes
__device__ __forceinline__ u64 wl_limb(u64 a, int src)
{
    const u64 v = __shfl(a, src & 63, 64);
    return (src >= 0 && src < 64) ? v : 0ull;
}

// a >> s (s >= 0), and whether any bit below s was set
__device__ __forceinline__ u64 wl_shr(u64 a, int s, bool *sticky)
{
    const int q = s >> 6, r = s & 63, lane = sts_lane();
    const u64 a0 = wl_limb(a, lane + q), a1 = wl_limb(a, lane + q + 1);
    const u64 low = lane < q ? a : (lane == q && r ? (a & ((1ull << r) - 1)) : 0ull);
    *sticky = __ballot(low != 0) != 0;
    return r ? (a0 >> r) | (a1 << (64 - r)) : a0;
}

// ceil(a * m / 2^s), m < 2^64
__device__ __forceinline__ u64 wl_mul_shr_ceil(u64 a, u64 m, int s)
{
    const u128 pr = (u128)a * m;
    const u64 hi_below = __shfl_up((u64)(pr >> 64), 1, 64);
    const u64 t = wl_add((u64)pr, sts_lane() > 0 ? hi_below : 0ull);
    bool sticky;
    const u64 q = wl_shr(t, s, &sticky);
    return sticky ? wl_add(q, sts_lane() == 0 ? 1ull : 0ull) : q;
}

// nearest binary64 (ties to even); the result is the same in every lane
__device__ inline double wl_to_double(u64 a)
{
    const u64 NZ = __ballot(a != 0);
    if (!NZ) return 0.0;
    const int top = 63 - __clzll((long long)NZ);
    const u64 L0 = wl_limb(a, top), L1 = wl_limb(a, top - 1), L2 = wl_limb(a, top - 2);
    const bool below = top >= 3 && (NZ & ((1ull << (top - 2)) - 1)) != 0;
    const int lz = __clzll((long long)L0);
    const int h = top * 64 + 63 - lz; // position of the top set bit
    if (h < 53) return ldexp((double)L0, -1074);
    const u64 hi = lz ? (L0 << lz) | (L1 >> (64 - lz)) : L0; // bit 63 = bit h
    const u64 lo = lz ? (L1 << lz) | (L2 >> (64 - lz)) : L1;
    const bool rest = below || (lz ? (L2 << lz) != 0 : L2 != 0);
    u64 mant = hi >> 11;
    const bool guard = (hi >> 10) & 1ull;
    const bool sticky = (hi & 0x3ffull) != 0 || lo != 0 || rest;
    int lsb = h - 52;
    if (guard && (sticky || (mant & 1ull))) {
        mant += 1;
        if (mant == (1ull << 53)) {
            mant >>= 1;
            lsb += 1;
        }
    }
    return ldexp((double)mant, lsb - 1074);
}

// Subset of the rank order still holding the cut: the terms of exponent e*
// whose rank key V has the high part vpre above bit vshift.
struct Sub {
    u64 cnt_before; // terms ranked before the subset
    u128 mb;        // their mantissa sum inside e* (units 2^(max(e*,1)-1075))
    u128 vpre;
    int vshift;
    u64 count;      // terms in the subset
};

__device__ inline void sub_load(Sub &s, const DevCtl *ctl)
{
    s.cnt_before = ctl->cnt_before;
    s.mb = make128(ctl->mb_lo, ctl->mb_hi);
    s.vpre = make128(ctl->vpre_lo, ctl->vpre_hi);
    s.vshift = ctl->vshift;
    s.count = ctl->sub_count;
}

__device__ inline void sub_store(const Sub &s, DevCtl *ctl)
{
    ctl->cnt_before = s.cnt_before;
    ctl->mb_lo = (u64)s.mb;
    ctl->mb_hi = (u64)(s.mb >> 64);
    ctl->vpre_lo = (u64)s.vpre;
    ctl->vpre_hi = (u64)(s.vpre >> 64);
    ctl->vshift = s.vshift;
    ctl->sub_count = s.count;
}

// bins in three arrays (count, mantissa sum >> 26, & (2^26 - 1)), in device
// memory that other workgroups wrote (agent loads) or in LDS
struct AgentBins {
    const u64 *h;
    __device__ __forceinline__ void operator()(u32 d, u64 &c, u128 &m) const
    {
        c = ld_agent(&h[d]);
        m = ((u128)ld_agent(&h[STS_NBIN + d]) << 26) + (u128)ld_agent(&h[2 * STS_NBIN + d]);
    }
};
struct WideBins {
    const u64 *h;
    __device__ __forceinline__ void operator()(u32 d, u64 &c, u128 &m) const
    {
        c = h[d];
        m = ((u128)h[STS_NBIN + d] << 26) + (u128)h[2 * STS_NBIN + d];
    }
};

// Pick the first digit (ascending = rank order) where the rule is met, over
// 2048 bins - bins(d, count, mass) - by a workgroup of NT threads, and narrow
// *sub to it. K, R: the rule (R all ones = no p-mass). Returns false if no
// digit qualifies. Four waves do the work, each thread on some neighbouring
// bins, and only the wave that holds the digit looks at single bins: the
// arithmetic of a workgroup that is alone on its CU costs its waves times the
// instructions (with two bins per thread of 16 waves and scans through LDS the
// pick of k_bkt_select took 6.1 us instead of 2.0). s_m, s_c: 4 entries.
template <int NT, typename BINS>
__device__ __forceinline__ bool pick_digit(const BINS &bins, u64 K, u128 R, int dw, Sub *sub, u128 *s_m, u64 *s_c, u32 *s_hit)
{
    constexpr int PT = NT < 256 ? NT : 256, PER = STS_NBIN / PT, LG = 3;
    static_assert(PER == 1 << LG, "a row of lanes takes a thread's bins");
    const int t = threadIdx.x, lane = sts_lane(), wv = __builtin_amdgcn_readfirstlane(t >> 6);
    // the subset as it is before this level (one thread narrows it after the barrier)
    const u64 cnt0 = sub->cnt_before;
    const u128 m0 = sub->mb;
    // met by the terms up to a point of the ranking (some of them in the subset)
    auto met = [&](u64 c, u128 m) { return c > 0 && ((K > 0 && cnt0 + c >= K) || m0 + m >= R); };
    u64 c = 0;
    u128 m = 0;
    if (t < PT) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            u64 ck;
            u128 mk;
            bins((u32)(PER * t + k), ck, mk);
            c += ck;
            m += mk;
        }
        c = wave_incl_scan(c);
        m = wave_incl_scan(m);
        if (lane == 63) {
            s_c[wv] = c;
            s_m[wv] = m;
        }
    }
    if (t == 0) *s_hit = 0;
    __syncthreads();
    // the wave, the lane and the bin that reach it first: the rule only grows
    // along the ranking
    if (t < PT) {
        const u64 tc = row_incl_scan(lane < PT / 64 ? s_c[lane] : 0ull);
        const u128 tm = row_incl_scan(lane < PT / 64 ? s_m[lane] : (u128)0);
        u64 cb = 0;
        u128 mb = 0;
        if (wv > 0) {
            cb = sts_readlane(tc, wv - 1);
            mb = sts_readlane(tm, wv - 1);
        }
        const u64 hits = __ballot(met(cb + c, mb + m));
        if (hits && !met(cb, mb)) { // uniform: this wave
            const int L = __builtin_ctzll(hits);
            if (L > 0) { // the terms before lane L
                cb += sts_readlane(c, L - 1);
                mb += sts_readlane(m, L - 1);
            }
            const u32 d = (u32)(PER * ((wv << 6) + L)) + (u32)(lane & (PER - 1));
            u64 ck;
            u128 mk;
            bins(d, ck, mk);
            u64 cs = ck;
            u128 ms = mk;
            cs += sts_dpp<0x111>(cs);
            ms += sts_dpp<0x111>(ms);
            cs += sts_dpp<0x112>(cs);
            ms += sts_dpp<0x112>(ms);
            cs += sts_dpp<0x114>(cs);
            ms += sts_dpp<0x114>(ms);
            const u64 first = __ballot(met(cb + cs, mb + ms)); // of lanes 0 to PER - 1; not 0
            if (lane == __builtin_ctzll(first)) {
                const u128 vpre = (sub->vpre << dw) | (u128)d;
                sub->cnt_before = cnt0 + cb + cs - ck;
                sub->mb = m0 + mb + ms - mk;
                sub->vpre = vpre;
                sub->vshift -= dw;
                sub->count = ck;
                *s_hit = 1;
            }
        }
    }
    __syncthreads();
    return *s_hit != 0;
}

// within-exponent rank key: ascending V = descending weight, then ascending key
__device__ __forceinline__ u128 rank_key(u64 wbits, u64 key)
{
    const u64 frac = wbits & ((1ull << 52) - 1);
    return ((u128)(((1ull << 52) - 1) - frac) << 64) | (u128)key;
}

__device__ __forceinline__ u64 mant_of_v(u128 v, int e)
{
    const u64 frac = ((1ull << 52) - 1) - (u64)(v >> 64);
    return e ? (frac | (1ull << 52)) : frac;
}


// ---------------------------------------------------------------------------
// level 1: one workgroup of NT threads. Thread t owns the NB = 2048 / NT
// exponent bins from 2047 - NB t down (descending weight order). The bins that
// hold candidates are listed in rank order in LDS, their mantissa sums as the
// limbs they take; four waves add the exact masses of a quarter of them each,
// limbs and carries apart, so that no bin waits for another's carries. One wave
// then has the total W and the p-mass target, finds with doubles the first bin
// where the rule may be met, and decides exactly from there. A chain of LDS
// and register latencies: 5.6 us in k_bkt_select, 8.4 when every bin's carries
// were resolved in turn.
// ---------------------------------------------------------------------------
// what the level-1 pick found, for the rest of the same workgroup
struct Level1Cut {
    int keep_all;
    int e;            // exponent field that holds the cut
    u64 total;        // candidates
    double W;
    u64 cnt, count;   // terms ranked before e's, and e's
    int in_window;    // the window holds the cut:
    u64 w_cnt, w_count, w_mb_lo, w_mb_hi; // terms ranked before its own, its own, and the mass in e before them
    u64 R_lo, R_hi;   // mass to reach inside e, in its units (all ones: off)
    u64 S[STS_NL];    // exact mass ranked before e's terms
};

template <int NT> struct Level1Smem {
    unsigned short e[STS_NBIN]; // the non-empty bins in rank order: exponent field,
    u64 c[STS_NBIN];   // count,
    // mantissa sum, as the three limbs that it takes from limb (unit bit / 64) on
    __attribute__((aligned(16))) u64 p[3][STS_NBIN];
    u32 scan[NT / 64];
    u64 bw[NT / 64], bk[NT / 64];
    u64 w[9];
    Sub sub;   // level 2 of a sampled window that holds the cut
    u32 fine, hit2;
    u64 R_lo, R_hi;
    u64 chunk[4][64]; // exact mass of each quarter of the bin list (a limb per lane)
    Level1Cut cut;
};

// the exponent bins in device memory
template <int NT> struct DeviceBins {
    u64 *h1;
    __device__ __forceinline__ void load(int, int e, u64 &c, u64 &hi, u64 &lo) const
    {
        c = h1[e];
        hi = h1[STS_NBIN + e];
        lo = h1[2 * STS_NBIN + e];
    }
    __device__ __forceinline__ void clear(int t) const
    {
        for (int i = t; i < 3 * STS_NBIN; i += NT) h1[i] = 0;
    }
};

// the same, the loads issued beforehand
template <int NT> struct EarlyBins : DeviceBins<NT> {
    u64 c[STS_NBIN / NT], hi[STS_NBIN / NT], lo[STS_NBIN / NT];
    __device__ __forceinline__ EarlyBins(u64 *h1) : DeviceBins<NT>{h1}
    {
#pragma unroll
        for (int k = 0; k < STS_NBIN / NT; ++k)
            DeviceBins<NT>::load(k, 2047 - STS_NBIN / NT * (int)threadIdx.x - k, c[k], hi[k], lo[k]);
    }
    __device__ __forceinline__ void load(int k, int, u64 &ck, u64 &hk, u64 &lk) const
    {
        ck = c[k];
        hk = hi[k];
        lk = lo[k];
    }
};

// predicted: 0 no window, 1 a window of the tiled passes, 2 one without level-2 bins, 3 a bucketed step
// whose histogram pass ran (no window; the slabs hold every candidate, or the side
// buffer, if the extraction pass fills it, is packed densely)
// bins: load(k, e, count, mantissa sum >> 26, & (2^26 - 1)) of exponent field e,
// the thread's k-th, and clear(t) by every thread when all are read
template <int NT, typename BINS>
__device__ __forceinline__ void pick_level1(const PassBufs &b, int groups, int peak_only, int predicted, Level1Smem<NT> &sm,
                            const BINS &bins)
{
    constexpr int NB = STS_NBIN / NT, NW = NT / 64;
    constexpr int NC = 4; // chunks of the bin list
    const int t = threadIdx.x;
    DevCtl *ctl = b.ctl;
    // the exponent of the window the histogram pass copied (predicted steps)
    const int w_mode = ctl->w_mode;
    const bool win = predicted == 1 || predicted == 2;
    const int e_w = win ? (w_mode ? ctl->e_w : ctl->e_pred) : -1;
    const int e_floor = predicted == 3 ? slab_floor(b, ctl->e_pred) : 0; // (read before the cut's is written)
    const int e_w2 = predicted == 2 ? (int)(ctl->w_lo >> 52) : -1; // (e_w itself as a rule)
    if (t < 9) sm.w[t] = 0;
    if (t == 0) sm.fine = 0;

    // own bins: every load issued before any is used
    u64 c[NB], hi[NB], lo[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int e = 2047 - NB * t - k;
        bins.load(k, e, c[k], hi[k], lo[k]);
    }
    // the per-workgroup peaks too (reduced below)
    constexpr int BPT = (STS_MAX_GROUPS + NT - 1) / NT;
    u64 bwv[BPT], bkv[BPT];
#pragma unroll
    for (int r = 0; r < BPT; ++r) {
        const int i = t + NT * r;
        bwv[r] = peak_only && i < groups ? b.best[i] : 0ull;
        bkv[r] = peak_only && i < groups ? b.best[STS_MAX_GROUPS + i] : ~0ull;
    }
    // the window sums of the histogram workgroups: count of candidates above
    // the window and mantissa sums of those in its exponent, then count and
    // sums of those inside it
    // (loaded whenever the pass predicted, before the control block says
    // whether a window was copied)
    // (predicted == 2: then count and sums of those inside it in the exponent below)
    u64 v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int fields = predicted == 2 ? 9 : 6;
    if (win) {
#pragma unroll
        for (int r = 0; r < STS_MAX_GROUPS / NT; ++r) { // every load issued before any is used
            const int i = t + NT * r;
            if (i < groups) {
#pragma unroll
                for (int f = 0; f < 9; ++f)
                    if (f < fields) v[f] += b.wpart[f * STS_MAX_GROUPS + i];
            }
        }
    }
    if (e_w >= 0) {
#pragma unroll
        for (int f = 0; f < 9; ++f)
            if (f < fields) v[f] = wave_incl_scan(v[f]); // (lane 63: the sum)
        __syncthreads(); // sm.w cleared
        if ((t & 63) == 63) {
#pragma unroll
            for (int f = 0; f < 9; ++f)
                if (f < fields && v[f]) atomicAdd((unsigned long long *)&sm.w[f], (unsigned long long)v[f]);
        }
    }
    // list the non-empty bins in rank order
    u32 nz = 0;
#pragma unroll
    for (int k = 0; k < NB; ++k) nz += c[k] ? 1u : 0u;
    u32 nbins;
    u32 at = block_excl_scan<u32, NT>(nz, sm.scan, &nbins);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        if (!c[k]) continue;
        sm.e[at] = (unsigned short)(2047 - NB * t - k);
        sm.c[at] = c[k];
        const u128 ms = ((u128)hi[k] << 26) + (u128)lo[k];
        const int off = unit_bit(2047 - NB * t - k) & 63;
        const u128 ml = ms << off;
        sm.p[0][at] = (u64)ml;
        sm.p[1][at] = (u64)(ml >> 64);
        sm.p[2][at] = off ? (u64)(ms >> 64) >> (64 - off) : 0ull;
        ++at;
    }
    // peak: reduce the per-workgroup bests (written by the identity pass of
    // sts_peak only)
    if (peak_only) {
        u64 bw = 0, bk = ~0ull;
#pragma unroll
        for (int r = 0; r < BPT; ++r) {
            const u64 w = bwv[r], k = bkv[r];
            if (w > bw || (w == bw && k < bk)) {
                bw = w;
                bk = k;
            }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const u64 ow = __shfl_xor(bw, d, 64);
            const u64 ok = __shfl_xor(bk, d, 64);
            if (ow > bw || (ow == bw && ok < bk)) {
                bw = ow;
                bk = ok;
            }
        }
        if ((t & 63) == 0) {
            sm.bw[t >> 6] = bw;
            sm.bk[t >> 6] = bk;
        }
    }
    __syncthreads();

    // this lane's limb of bin j
    auto piece = [&](u32 j) {
        const u32 k = (u32)(t & 63) - ((u32)unit_bit((int)sm.e[j]) >> 6);
        return k < 3u ? sm.p[k][j] : 0ull;
    };
    // exact sum of bins j0 to j1: limbs and their carries are added up
    // separately, and the carries resolved once at the end
    auto add_bins = [&](u64 start, u32 j0, u32 j1) {
        u64 acc = start;
        u32 carry = 0;
#pragma unroll 4
        for (u32 j = j0; j < j1; ++j) {
            const u64 v = piece(j);
            acc += v;
            carry += acc < v ? 1u : 0u;
        }
        const u32 in = __shfl_up(carry, 1, 64);
        return wl_add(acc, (t & 63) ? (u64)in : 0ull);
    };
    // in four chunks, one wave each
    const u32 chunk = (nbins + NC - 1) / NC;
    if (t < 64 * NC) {
        const int q = t >> 6;
        const u32 j0 = (u32)q * chunk < nbins ? (u32)q * chunk : nbins, j1 = j0 + chunk < nbins ? j0 + chunk : nbins;
        sm.chunk[q][t & 63] = add_bins(0, j0, j1);
    }
    __syncthreads();

    if (t < 64) { // one wave: the total, the target and the cut's bin
        const int lane = t;
        u64 W = 0;
#pragma unroll
        for (int q = 0; q < NC; ++q) W = wl_add(W, sm.chunk[q][lane]);
        // the counts, and the masses as doubles in units of the first bin's
        // lowest limb (a total off by less than 2^-40 of it)
        auto approx = [&](u32 j) {
            if (j >= nbins) return 0.0;
            const int sh = (unit_bit((int)sm.e[j]) >> 6) - (unit_bit((int)sm.e[0]) >> 6); // <= 0
            const double m = (double)sm.p[0][j] + 0x1p64 * ((double)sm.p[1][j] + 0x1p64 * (double)sm.p[2][j]);
            return sh < -15 ? 0.0 : ldexp(m, 64 * sh);
        };
        const double p = ctl->p;
        const bool p_on = p > 0.0 && p < 1.0, by_mass = p_on && !peak_only;
        u64 total_c = 0;
        double total_m = 0.0;
        for (u32 j0 = 0; j0 < nbins; j0 += 64) {
            const u32 j = j0 + (u32)lane;
            total_c += sts_readlane(wave_incl_scan(j < nbins ? sm.c[j] : 0ull), 63);
            if (by_mass) total_m += sts_readlane(wave_incl_scan(approx(j)), 63);
        }
        const double Wd = wl_to_double(W);
        if (peak_only) {
            if (lane == 0) {
                ctl->cand_all = total_c;
                ctl->peak_W = Wd;
                u64 w = sm.bw[0], k = sm.bk[0];
                for (int i = 1; i < NW; ++i)
                    if (sm.bw[i] > w || (sm.bw[i] == w && sm.bk[i] < k)) {
                        w = sm.bw[i];
                        k = sm.bk[i];
                    }
                ctl->peak_key = k;
                ctl->peak_w = (w >> 63) ? __longlong_as_double((long long)(w & ~(1ull << 63))) : 0.0;
            }
        } else {
            const u64 K = ctl->K;
            // p-mass target T = ceil(p * W), exactly
            u64 T = 0;
            if (p_on) {
                const u64 pb = sts_dbits(p);
                const u64 pe = pb >> 52, pf = pb & ((1ull << 52) - 1);
                const u64 pm = pe ? (pf | (1ull << 52)) : pf;
                const int sh = pe ? (int)(1075 - pe) : 1074;
                T = wl_mul_shr_ceil(W, pm, sh);
            }
            if (lane < STS_NL) ctl->T.l[lane] = T;
            if (lane == 0) {
                ctl->cand_all = total_c;
                ctl->W = Wd;
                ctl->n_cand = total_c;
                ctl->tot_steps += 1;
                ctl->tot_updates += *b.n_in;
                ctl->tot_cand += total_c;
            }
            // after the histogram pass of a bucketed step: no more candidates than K
            // are no cut (of the least of them, which changes nothing)
            const bool uncut = predicted == 3 && !p_on && total_c <= K;
            // The first bin in rank order where the rule is met: the first
            // that meets it on the count or may meet it on the mass, judged by
            // doubles (error far below the margin); from there on exactly
            const double T_low = p * total_m * (1.0 - 0x1p-30);
            u32 hit = nbins;
            u64 cnt = 0;
            double m0 = 0.0;
            for (u32 j0 = 0; j0 < nbins && hit == nbins && !uncut; j0 += 64) {
                const u32 j = j0 + (u32)lane;
                const u64 cj = j < nbins ? sm.c[j] : 0ull;
                const u64 ci = cnt + wave_incl_scan(cj);
                const double mi = p_on ? m0 + wave_incl_scan(approx(j)) : 0.0;
                const u64 may = __ballot(j < nbins && ((K > 0 && ci >= K) || (p_on && mi >= T_low)));
                const int L = may ? __builtin_ctzll(may) : 63;
                if (may) hit = j0 + (u32)L;
                cnt = sts_readlane(may ? ci - cj : ci, L);
                m0 = sts_readlane(mi, L);
            }
            u64 S = 0;
            if (hit < nbins) {
                u32 j0 = 0;
                for (int q = 0; q < NC && j0 + chunk <= hit; ++q, j0 += chunk) S = wl_add(S, sm.chunk[q][lane]);
                S = add_bins(S, j0 < hit ? j0 : hit, hit);
            }
            for (;; ++hit) {
                if (hit >= nbins) {
                    hit = 0xffffffffu;
                    break;
                }
                const u64 inc = wl_add(S, piece(hit));
                if ((K > 0 && cnt + sm.c[hit] >= K) || (p_on && wl_cmp(inc, T) >= 0)) break;
                S = inc;
                cnt += sm.c[hit];
            }
            if (lane == 0) {
                sm.cut.keep_all = hit == 0xffffffffu;
                sm.cut.total = total_c;
                sm.cut.W = Wd;
            }
            if (hit == 0xffffffffu) {
                if (lane == 0) {
                    ctl->keep_all = 1;
                    ctl->dropped = 0;
                    ctl->L = total_c;
                    ctl->scale = 1.0;
                    ctl->S = Wd;
                    ctl->frac = 1.0;
                    ctl->level = 1;
                    ctl->pred_hit = 0;
                    ctl->e_pred = -1;
                }
            } else {
                const int e = (int)sm.e[hit];
                const int ub = unit_bit(e);
                // does the copied window hold the cut? Exactly when the rule is
                // not met through the candidates above it and is met through it
                bool in_window = false;
                u64 ca = 0, cw = 0;
                u128 ma = 0;
                if (e == e_w) {
                    // the histogram pass counted every candidate above the window;
                    // those in exponents above e are the cnt ranked before this bin
                    ca = sm.w[0] - cnt;
                    cw = sm.w[3];
                    ma = ((u128)sm.w[1] << 26) + (u128)sm.w[2];
                    const u128 mw = ((u128)sm.w[4] << 26) + (u128)sm.w[5];
                    const u64 Sa = wl_add(S, wl_piece((u64)ma, (u64)(ma >> 64), ub));
                    const bool met_a = (K > 0 && cnt + ca >= K) || (p_on && wl_cmp(Sa, T) >= 0);
                    const u64 Sw = wl_add(Sa, wl_piece((u64)mw, (u64)(mw >> 64), ub));
                    const bool met_w = (K > 0 && cnt + ca + cw >= K) || (p_on && wl_cmp(Sw, T) >= 0);
                    in_window = !met_a && met_w;
                } else if (predicted == 2 && e == e_w2) { // the window's part in the exponent below
                    cw = sm.w[6];
                    const u128 mw = ((u128)sm.w[7] << 26) + (u128)sm.w[8];
                    const u64 Sw = wl_add(S, wl_piece((u64)mw, (u64)(mw >> 64), ub));
                    in_window = (K > 0 && cnt + cw >= K) || (p_on && wl_cmp(Sw, T) >= 0);
                }
                // remaining mass to reach inside the bin, in its units (rounded up)
                u64 R_lo = ~0ull, R_hi = ~0ull;
                if (p_on) {
                    bool sticky;
                    const u64 q = wl_shr(wl_sub(T, S), ub, &sticky);
                    const bool over = __ballot(lane >= 2 && q != 0) != 0;
                    u128 r = ((u128)__shfl(q, 1, 64) << 64) | (u128)__shfl(q, 0, 64);
                    if (!over) {
                        if (sticky) r += 1;
                        if (r != 0 || !sticky) {
                            R_lo = (u64)r;
                            R_hi = (u64)(r >> 64);
                        }
                    }
                }
                if (lane < STS_NL) {
                    ctl->S_excl.l[lane] = S;
                    sm.cut.S[lane] = S;
                }
                if (lane == 0) {
                    sm.cut.e = e;
                    sm.cut.cnt = cnt;
                    sm.cut.count = sm.c[hit];
                    sm.cut.in_window = in_window;
                    sm.cut.w_cnt = cnt + ca;
                    sm.cut.w_count = cw;
                    sm.cut.w_mb_lo = (u64)ma;
                    sm.cut.w_mb_hi = (u64)(ma >> 64);
                    sm.cut.R_lo = R_lo;
                    sm.cut.R_hi = R_hi;
                }
                if (lane == 0 && in_window && w_mode && predicted == 1) {
                    // the histogram pass binned this window for level 2: the
                    // whole workgroup picks its digit below
                    sm.fine = 1;
                    sm.sub.cnt_before = cnt + ca;
                    sm.sub.mb = ma;
                    sm.sub.vpre = 0;
                    sm.sub.vshift = 116;
                    sm.sub.count = cw;
                    sm.R_lo = R_lo;
                    sm.R_hi = R_hi;
                }
                if (lane == 0) {
                    ctl->keep_all = 0;
                    ctl->pred_hit = in_window ? 1 : 0;
                    ctl->e_pred = e;
                    ctl->e_star = e;
                    ctl->cnt_before = in_window ? cnt + ca : cnt;
                    ctl->sub_count = in_window ? cw : sm.c[hit];
                    ctl->mb_lo = in_window ? (u64)ma : 0;
                    ctl->mb_hi = in_window ? (u64)(ma >> 64) : 0;
                    ctl->level = 1;
                    ctl->R_lo = R_lo;
                    ctl->R_hi = R_hi;
                }
            }
            if (lane == 0) {
                ctl->w2_mode = predicted == 1 && w_mode; // the histogram pass binned the window for level 2
                ctl->w_mode = 0;                     // a window serves one step
                if (predicted == 3) {
                    const bool every = b.keep && !ld_agent(&ctl->w_over) &&
                                       (hit != 0xffffffffu ? (int)sm.e[hit] >= e_floor : e_floor == 0);
                    ctl->slab_all = every;
                    ctl->w_over = 0;
                    ctl->need_full = 0;
                    // else the extraction pass packs its candidates densely
                    if (hit != 0xffffffffu && !every) {
                        ctl->side_dense = 1;
                        ctl->side_n = 0;
                    }
                }
                ctl->l2_done = 0;
            }
        }
    }
    __syncthreads();
    bins.clear(t);
    if (sm.fine) { // uniform
        // level 2 from the window's bins (the side pass then has nothing to
        // do); the bin lists above are done with, so their LDS serves the pick
        const u128 R = make128(sm.R_lo, sm.R_hi);
        u128 *s_m = reinterpret_cast<u128 *>(sm.p[0]);
        u64 *s_c2 = sm.p[1];
        const bool ok = pick_digit<NT>(AgentBins{b.h2w}, ctl->K, R, 11, &sm.sub,
                                        s_m, s_c2, &sm.hit2);
        if (ok && t <= STS_SUB_REGIONS) st_agent(&b.sub_cnt[t * 32], 0u);
        if (t == 0) {
            if (ok) {
                sub_store(sm.sub, ctl);
                ctl->level = 2;
                ctl->l2_done = 1;
            } else {
                atomicOr(&ctl->flags, STS_F_UNRESOLVED);
            }
        }
        for (int i = t; i < 3 * STS_NBIN; i += NT) st_agent(&b.h2w[i], 0ull);
    }
}

// ---------------------------------------------------------------------------
// Last levels: narrow `sub` by 11-bit digits of the rank key V until at most
// STS_FINAL_SORT terms are left, then find the exact cut among them.
// each(vshift, vpre, keyed, f) calls f(V) for every term of the subset whose V
// lies under the prefix (all threads take part; V's key half may be 0 unless
// keyed). raw: STS_NBIN * 24 bytes of LDS, or THIN_BINS * 12 when there are so few terms
// (below 2^22) that 64 bits hold a bin's sum of the 41 mantissa bits that the
// first level leaves open; cleared: the caller has zeroed it.
// ---------------------------------------------------------------------------
struct CutSmem {
    u128 m[1024 / 64];
    u64 c[1024 / 64];
    u32 hit, n;
    u32 rank[STS_FINAL_SORT]; // of the last terms
    u64 mass[STS_FINAL_SORT];
    u64 thr_w, thr_k;  // the cut's term
    u64 mk_lo, mk_hi;  // mantissa sum ranked up to it inside its exponent
    u64 L;
    double scale;
    int dropped;
};

// mantissa bits shared by the terms of exponent e whose first digit is d
__device__ __forceinline__ u64 digit_mant(u32 d, int e)
{
    return ((u64)(2047u - d) << 41) | (e ? 1ull << 52 : 0ull);
}

constexpr u64 LOW41 = (1ull << 41) - 1;

// LDS places of the thin bins: one free per eight, since a thread picks among
// eight neighbouring bins
constexpr int THIN_BINS = STS_NBIN + STS_NBIN / 8;
__device__ __forceinline__ u32 thin_at(u32 d) { return d + (d >> 3); }

// bins of one level: sums of the low 41 mantissa bits, and counts; the high
// bits come from the bin (first level) or are common to the subset
struct ThinBins {
    const u64 *low;
    const u32 *cnt;
    int e;
    bool first;
    u64 high;
    __device__ __forceinline__ void operator()(u32 d, u64 &c, u128 &m) const
    {
        const u32 n = cnt[thin_at(d)];
        c = n;
        // (below 2^22 terms: the first level's product, in units of 2^41, fits 64 bits)
        const u128 top = first ? (u128)((u64)((e ? 4095u : 2047u) - d) * n) << 41 : (u128)high * n;
        m = top + (u128)low[thin_at(d)];
    }
};

// A subset of more terms than this after a level is one of equal weights as a
// rule. At 2^21 equal weights k_final took 67 ms when every lane added for
// itself, 23 ms so.
constexpr u64 TIES = 4096;

// what a level's pass does with every term
template <bool THIN> struct Binner {
    u64 *h;
    u32 *hc;
    int shift, dw, e;
    bool many; // the subset is still large after a level
    __device__ __forceinline__ void operator()(const u128 v) const
    {
        const u32 d = (u32)((v >> shift) & (u128)((1u << dw) - 1));
        const u64 mant = mant_of_v(v, e);
        if (THIN) {
            atomicAdd((unsigned long long *)&h[thin_at(d)], mant & LOW41);
            atomicAdd(&hc[thin_at(d)], 1u);
        } else {
            u64 n = 1;
            if (many) { // uniform: equal weights as a rule, which would queue on one bin; one lane adds for all
                const u64 here = __ballot(true);
                if (__ballot(d == (u32)__builtin_amdgcn_readfirstlane((int)d) && mant == sts_firstlane(mant)) == here) {
                    if (sts_lanes_below(here) != 0) return;
                    n = (u64)__popcll(here);
                }
            }
            atomicAdd((unsigned long long *)&h[d], n);
            atomicAdd((unsigned long long *)&h[STS_NBIN + d], (mant >> 26) * n);
            atomicAdd((unsigned long long *)&h[2 * STS_NBIN + d], (mant & ((1ull << 26) - 1)) * n);
        }
    }
    // the same of a weight at the first level (shift 105, 11 bits)
    __device__ __forceinline__ void first(u64 w) const
    {
        static_assert(THIN, "thin bins");
        const u32 d = thin_at(2047u - ((u32)(w >> 41) & 2047u));
        atomicAdd((unsigned long long *)&h[d], w & LOW41);
        atomicAdd(&hc[d], 1u);
    }
};

template <int NT, bool THIN, typename E>
__device__ __forceinline__ bool narrow_cut(E &&each, int e, u64 K, u128 R, Sub &sub, unsigned char *raw, CutSmem &sm, u32 enough,
                           bool cleared = false)
{
    const int t = threadIdx.x;
    u64 *h = reinterpret_cast<u64 *>(raw);
    u32 *hc = reinterpret_cast<u32 *>(h + THIN_BINS);
    while (sub.count > enough && sub.vshift > 0) {
        const int vshift = sub.vshift;
        const int dw = vshift < 11 ? vshift : 11;
        const u128 vpre = sub.vpre;
        if (!cleared) {
            for (int i = t; i < (THIN ? THIN_BINS * 3 / 2 : 3 * STS_NBIN); i += NT) h[i] = 0;
            __syncthreads();
        }
        cleared = false;
        each(vshift, vpre, vshift - dw < 64, Binner<THIN>{h, hc, vshift - dw, dw, e, sub.count > TIES});
        __syncthreads();
        bool ok;
        if (THIN) {
            const bool first = vshift == 116;
            const u64 high = first ? 0ull : digit_mant((u32)(vpre >> (105 - vshift)), e);
            ok = pick_digit<NT>(ThinBins{h, hc, e, first, high}, K, R, dw, &sub, sm.m, sm.c, &sm.hit);
        } else {
            ok = pick_digit<NT>(WideBins{h}, K, R, dw, &sub, sm.m, sm.c, &sm.hit);
        }
        if (!ok) return false;
    }
    return true;
}

// the cut among the m <= STS_FINAL_SORT terms listed in sv (a handful as a
// rule): every term counts and weighs the ones before it by itself; their
// mantissas add up below 2^63. Returns this thread's rank (m or more: no term)
// The threads of a term share the comparisons (its partial sums meet in LDS).
template <int NT> __device__ __forceinline__ u32 rank_cut(const u128 *sv, u32 m, int e, u64 K, u128 R, const Sub &sub, CutSmem &sm)
{
    constexpr u32 PARTS = NT / STS_FINAL_SORT;
    static_assert(PARTS >= 1 && NT % STS_FINAL_SORT == 0, "whole parts");
    const u32 t = threadIdx.x, i = t % STS_FINAL_SORT, part = t / STS_FINAL_SORT;
    if (t < STS_FINAL_SORT) {
        sm.rank[t] = 0;
        sm.mass[t] = 0;
    }
    __syncthreads();
    if (i < m) {
        const u128 v = sv[i];
        u32 rank = 0;
        u64 mass = 0; // of the terms up to this one
        for (u32 j = part; j < m; j += PARTS) {
            const u128 o = sv[j];
            rank += o < v ? 1u : 0u;
            mass += o <= v ? mant_of_v(o, e) : 0ull;
        }
        if (rank) atomicAdd(&sm.rank[i], rank);
        if (mass) atomicAdd((unsigned long long *)&sm.mass[i], (unsigned long long)mass);
    }
    __syncthreads();
    const u32 rank = t < m ? sm.rank[t] : ~0u;
    const u64 mass = t < m ? sm.mass[t] : 0ull;
    const bool met = t < m && ((K > 0 && sub.cnt_before + rank + 1 >= K) || sub.mb + (u128)mass >= R);
    if (met) atomicMin(&sm.hit, rank);
    __syncthreads();
    if (met && rank == sm.hit) {
        const u128 v = sv[t], mk = sub.mb + (u128)mass;
        sm.thr_w = ((u64)e << 52) | (((1ull << 52) - 1) - (u64)(v >> 64));
        sm.thr_k = (u64)v;
        sm.mk_lo = (u64)mk;
        sm.mk_hi = (u64)(mk >> 64);
        sm.L = sub.cnt_before + rank + 1;
    }
    __syncthreads();
    return rank;
}

// one wave: the kept mass, the scale and the statistics (S_excl: the exact
// mass ranked before exponent e's part, one limb per entry)
__device__ __forceinline__ void finish_cut(DevCtl *ctl, CutSmem &sm, int e, const u64 *S_excl, u64 ncand, double W,
                                           double l10)
{
    const int lane = sts_lane();
    const u64 x = lane < STS_NL ? S_excl[lane] : 0ull;
    const double Sd = wl_to_double(wl_add(x, wl_piece(sm.mk_lo, sm.mk_hi, unit_bit(e))));
    if (lane == 0) {
        const int dropped = sm.L < ncand;
        const double scale = dropped ? 1.0 / sqrt(Sd) : 1.0;
        sm.dropped = dropped;
        sm.scale = scale;
        ctl->L = sm.L;
        ctl->thr_wbits = sm.thr_w;
        ctl->thr_key = sm.thr_k;
        ctl->dropped = dropped;
        ctl->S = Sd;
        ctl->scale = scale;
        const double frac_kept = Sd / W;
        ctl->frac = frac_kept;
        if (dropped) ctl->log10_cum = l10 + log10(frac_kept);
    }
}

// all of it, up to the cut's term in sm (false: the cut could not be resolved,
// an internal inconsistency); finish_cut by one wave follows
template <int NT, bool THIN, typename E>
__device__ __forceinline__ bool resolve_cut(E &&each, int e, u64 K, u128 R, Sub &sub, unsigned char *raw, CutSmem &sm)
{
    if (!narrow_cut<NT, THIN>(each, e, K, R, sub, raw, sm, STS_FINAL_SORT)) return false;
    u128 *sv = reinterpret_cast<u128 *>(raw);
    const int vshift = sub.vshift;
    const u128 vpre = sub.vpre;
    if (threadIdx.x == 0) {
        sm.n = 0;
        sm.hit = 0xffffffffu;
    }
    __syncthreads();
    each(vshift, vpre, true, [&](const u128 v) {
        const u32 slot = atomicAdd(&sm.n, 1u);
        if (slot < STS_FINAL_SORT) sv[slot] = v;
    });
    __syncthreads();
    const u32 m = sm.n;
    if (m == 0 || m > STS_FINAL_SORT) return false;
    (void)rank_cut<NT>(sv, m, e, K, R, sub, sm);
    return sm.hit != 0xffffffffu;
}

} // namespace sts_select
