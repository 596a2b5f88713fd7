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
// several rounds, each with the groups whose second hash has one prefix; the
// prefix grows until the round fits, so any distribution of keys is handled.
#pragma once
#include "group_impl.h"

namespace sts_bucket {

using namespace sts_group;

constexpr int BW = STS_WG / 64;    // waves of a workgroup, each with a share of its own
constexpr int BW_CAP = 320;        // terms of a share staged at once
constexpr int BW_SLOTS = 512;      // hash slots of a wave
constexpr int BW_ROUNDS = BW_CAP / 64;
constexpr u32 BW_BINNED = 640;     // larger shares bypass the LDS bins (their sums are bounded by this)
constexpr int BW_FLUSH = 16;       // tiles between flushes of the LDS bins

template <typename AT> struct BktSmem {
    AT amp[BW][BW_CAP];
    u64 key[BW][BW_CAP];
    unsigned long long slot[BW][BW_SLOTS]; // a group: the staged index + 1 of its member j at bit 16 j
    unsigned short lead[BW][BW_CAP];       // slots of the groups, in the order they were opened
};

// orders a wave's own LDS accesses (which the hardware performs in order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ u32 uni(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }

// the four runs of a wave's share (in scalar registers)
struct Share {
    u32 o0, o1, o2, o3; // first term of each run, less its start in the flat index
    u32 p1, p2, p3, n;  // starts of runs 1..3 in the flat index; terms in all
};

__device__ __forceinline__ Share load_share(const BktPlan &p, const uint2 *__restrict__ bd, u32 tile, int wv)
{
    const u32 lane = (u32)sts_lane();
    const u32 bucket = bkt_rep(p, tile) ^ bkt_comb(p, (lane & 3u) | ((u32)wv << 2));
    const uint2 d = bd[bucket];
    u32 beg[4], cnt[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        beg[i] = (u32)__builtin_amdgcn_readlane((int)d.x, i);
        cnt[i] = (u32)__builtin_amdgcn_readlane((int)d.y, i) - beg[i];
    }
    Share s;
    s.p1 = cnt[0];
    s.p2 = s.p1 + cnt[1];
    s.p3 = s.p2 + cnt[2];
    s.n = s.p3 + cnt[3];
    s.o0 = beg[0];
    s.o1 = beg[1] - s.p1;
    s.o2 = beg[2] - s.p2;
    s.o3 = beg[3] - s.p3;
    return s;
}

__device__ __forceinline__ u32 share_at(const Share &s, u32 j)
{
    u32 o = j < s.p1 ? s.o0 : s.o1;
    o = j < s.p2 ? o : s.o2;
    o = j < s.p3 ? o : s.o3;
    return o + j;
}

__device__ __forceinline__ u32 slot_hash(u64 rest)
{
    return ((u32)rest * 0x9e3779b1u + (u32)(rest >> 32) * 0x85ebca6bu) >> 23; // BW_SLOTS = 2^9
}

// stage the terms of the share (all of them, or those whose second hash has
// the prefix `pre` of `depth` bits); returns how many there are (more than
// BW_CAP: not staged)
template <typename AT>
__device__ __forceinline__ u32 stage_all(BktSmem<AT> &s, const Share &t, int wv, const u64 *__restrict__ keys,
                                         const AT *__restrict__ amps)
{
    const u32 lane = (u32)sts_lane();
    u64 kk[BW_ROUNDS];
    AT aa[BW_ROUNDS];
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        if (j < t.n) {
            const u32 at = share_at(t, j);
            kk[r] = keys[at];
            aa[r] = amps[at];
        }
    }
#pragma unroll
    for (int r = 0; r < BW_ROUNDS; ++r) {
        const u32 j = (u32)r * 64 + lane;
        if (j < t.n) {
            s.key[wv][j] = kk[r];
            s.amp[wv][j] = aa[r];
        }
    }
    return t.n;
}

template <typename AT>
__device__ __noinline__ u32 stage_part(BktSmem<AT> &s, const Share &t, int wv, const u64 *__restrict__ keys,
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
        const u64 m = __ballot(keep);
        const u32 pos = count + sts_lanes_below(m);
        if (keep && pos < BW_CAP) {
            s.key[wv][pos] = k;
            s.amp[wv][pos] = amps[at];
        }
        count += (u32)__popcll(m);
    }
    return count;
}

// group the `cnt` staged terms: every group gets a slot (open addressing on
// the masked key) that lists its members; returns the number of groups, their
// slots in s.lead
template <typename AT, int M>
__device__ __forceinline__ u32 build_groups(BktSmem<AT> &s, const GateArg &g, int wv, u32 cnt)
{
    const u32 lane = (u32)sts_lane();
    const u64 nm = g.notmask;
    u32 ngroups = 0;
    for (u32 r0 = 0; r0 < cnt; r0 += 64) {
        const u32 j = r0 + lane;
        bool todo = j < cnt, opened = false;
        u32 sl = 0;
        u64 rest = 0;
        unsigned long long mine = 0;
        if (todo) {
            const u64 key = s.key[wv][j];
            rest = key & nm;
            sl = slot_hash(rest);
            mine = (unsigned long long)(j + 1) << (16 * extract_bits<M>(key, g));
        }
        while (__ballot(todo)) {
            if (todo) {
                const unsigned long long old = atomicCAS(&s.slot[wv][sl], 0ull, mine);
                if (old == 0) {
                    opened = true;
                    todo = false;
                } else {
                    // any member tells the group
                    const int f = (__ffsll((long long)old) - 1) & ~15;
                    const u32 o = (u32)((old >> f) & 0xffffu) - 1u;
                    if ((s.key[wv][o] & nm) == rest) {
                        atomicOr(&s.slot[wv][sl], mine);
                        todo = false;
                    } else {
                        sl = (sl + 1) & (BW_SLOTS - 1);
                    }
                }
            }
        }
        const u64 m = __ballot(opened);
        if (opened) s.lead[wv][ngroups + sts_lanes_below(m)] = (unsigned short)sl;
        ngroups += (u32)__popcll(m);
    }
    wave_sync();
    return ngroups;
}

// body(G) for the groups of a share, one per lane (lanes without one have
// G.present = 0); every lane of the wave takes part
template <typename AT, int M, typename F>
__device__ __forceinline__ void share_groups(BktSmem<AT> &s, const GateArg &g, const Share &t, int wv,
                                             const u64 *__restrict__ keys, const AT *__restrict__ amps, F &&body)
{
    const u32 lane = (u32)sts_lane();
    int depth = 0;
    u64 pre = 0;
    if (t.n > BW_CAP)
        while ((t.n >> depth) > BW_CAP * 3 / 4) ++depth;
    for (;;) {
        u32 cnt;
        if (depth == 0) {
            cnt = stage_all<AT>(s, t, wv, keys, amps);
        } else {
            cnt = uni(stage_part<AT>(s, t, wv, keys, amps, g.notmask, depth, pre));
            if (cnt > BW_CAP) { // split the prefix (at 64 bits a part is one group)
                ++depth;
                pre <<= 1;
                continue;
            }
        }
        wave_sync();
        const u32 ng = build_groups<AT, M>(s, g, wv, cnt);
#pragma unroll 1
        for (u32 r0 = 0; r0 < ng; r0 += 64) {
            const u32 q = r0 + lane;
            Group<AT, M> G;
            G.present = 0;
            G.rest = 0;
            group_clear<AT, M>(G);
            if (q < ng) {
                const u32 sl = s.lead[wv][q];
                const unsigned long long w = s.slot[wv][sl];
                s.slot[wv][sl] = 0; // free again for the next part
                const int f = (__ffsll((long long)w) - 1) & ~15;
                G.rest = s.key[wv][(u32)((w >> f) & 0xffffu) - 1u] & g.notmask;
#pragma unroll
                for (int j = 0; j < (1 << M); ++j) {
                    const u32 i = (u32)((w >> (16 * j)) & 0xffffu);
                    if (i) {
                        G.v[j] = s.amp[wv][i - 1];
                        G.present |= 1u << j;
                    }
                }
            }
            body(G);
        }
        wave_sync();
        if (depth == 0) break;
        ++pre;
        if (depth < 64 && pre == (1ull << depth)) break;
        if (depth == 64 && pre == 0) break;
    }
}

template <typename AT> __device__ __forceinline__ void clear_slots(BktSmem<AT> &s)
{
    unsigned long long *p = &s.slot[0][0];
    for (int i = threadIdx.x; i < BW * BW_SLOTS; i += STS_WG) p[i] = 0;
}

__device__ __forceinline__ u32 bkt_tiles(const BktPlan &p) { return 1u << (p.hb - STS_BKT_DIMS); }

// ---------------------------------------------------------------------------
// histogram pass: exponent histogram with exact mantissa sums of all new
// weights; the window's candidates and those above it to the wave's slab (2^
// side_slab_shift entries: the window's from its start, those above from its
// end); a slab that is too small marks the window as missed. Persistent grid.
// ---------------------------------------------------------------------------
template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG, 3) k_bkt_hist(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    __shared__ BktSmem<AT> s;
    __shared__ u64 s_hi[TT_SLOTS], s_lo[TT_SLOTS];
    __shared__ u64 s_wacc[6];
    __shared__ u64 s_w2hi[TT_W2], s_w2lo[TT_W2];
    clear_slots<AT>(s);
    for (int i = threadIdx.x; i < TT_SLOTS; i += STS_WG) {
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
    for (int i = threadIdx.x; i < TT_W2; i += STS_WG) {
        s_w2hi[i] = 0;
        s_w2lo[i] = 0;
    }
    if (threadIdx.x < 6) s_wacc[threadIdx.x] = 0;
    DevCtl *ctl = b.ctl;
    const u64 *keys = b.keys;
    const AT *amps = (const AT *)b.amps;
    const u32 ntiles = bkt_tiles(g.bkt);
    int e_w = -1;
    u64 w_lo = 0, w_hi = 0;
    bool fine = false;
    if (b.predict) {
        if (ctl->w_mode) {
            e_w = ctl->e_w;
            w_lo = ctl->w_lo;
            w_hi = ctl->w_hi;
            fine = true;
        } else if (ctl->e_pred >= 0) {
            e_w = ctl->e_pred;
            w_lo = (u64)e_w << 52;
            w_hi = w_lo | ((1ull << 52) - 1);
        }
    }
    const bool predict = e_w >= 0;
    const u32 d_lo = (u32)((((1ull << 52) - 1) - (w_hi & ((1ull << 52) - 1))) >> 41);
    const u32 d_top = 2047u - d_lo;
    // the window's edges are multiples of 2^47 in the weight bits: the high
    // words decide
    const u32 wL = (u32)(w_lo >> 32), wH = (u32)((w_hi + 1) >> 32), wE1 = (u32)(e_w + 1) << 20;
    u64 ma = 0, mw = 0;
    const int shift = b.slab_shift;
    if (predict && blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->side_dense = 0;
        ctl->side_ntiles = (u64)ntiles << 2;
        ctl->side_slab_shift = shift;
        ctl->side_spt_log2 = 2;
    }
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int copy = (int)(threadIdx.x % TT_HCOPIES);
    const int e_ref = predict ? e_w : (ctl->e_pred >= 0 ? ctl->e_pred : TT_EBASE + 116);
    const int hot_lo = e_ref - (TT_HOT - 4);
    __syncthreads();
    int since_flush = 0;
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (since_flush == BW_FLUSH) {
            // a tile adds at most 4 * BW_BINNED * 4 candidates to the bins
            __syncthreads();
            flush_bins(b, s_hi, s_lo, hot_lo);
            if (predict) flush_window(s_wacc, ma, mw);
            if (fine) flush_w2(b, s_w2hi, s_w2lo, d_lo);
            since_flush = 0;
            __syncthreads();
        }
        ++since_flush;
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        const u32 sl = (tile << 2) + (u32)wv;
        const u64 slab = (u64)sl << shift;
        const u32 room = 1u << shift;
        const bool direct = sh.n > BW_BINNED;
        u64 *const sk = b.side_key + slab;
        u64 *const sw = b.side_w + slab;
        AT *const sa = (AT *)b.side_amp + slab;
        u32 c_in = 0, c_ab = 0, c_all = 0;
        bool fits = true;
        share_groups<AT, M>(s, g, sh, wv, keys, amps, [&](const Group<AT, M> &G) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT o = group_out<AT, M>(g, G, i);
                const bool cand = G.present && nonzero(o);
                const u64 wb = weight_bits(o);
                const int e_ = (int)(wb >> 52);
                bool ab = false, inw = false;
                if (cand) {
                    const u64 mant = sts_mant(wb);
                    if (predict) {
                        const u32 hw = (u32)(wb >> 32);
                        ab = hw >= wH;
                        inw = hw >= wL && !ab;
                        mw += inw ? mant : 0ull;
                        ma += (ab && hw < wE1) ? mant : 0ull;
                        if (fine && inw) {
                            const u32 rel = d_top - ((hw >> 9) & 2047u);
                            if (rel >= (u32)TT_W2) { // outside the window's bins: cannot happen; fail the step
                                atomicOr(&ctl->flags, STS_F_UNRESOLVED);
                            } else if (direct) {
                                const u32 d = d_lo + rel;
                                atomicAdd(&b.h2w[d], 1ull);
                                atomicAdd(&b.h2w[STS_NBIN + d], mant >> 26);
                                atomicAdd(&b.h2w[2 * STS_NBIN + d], mant & ((1ull << 26) - 1));
                            } else {
                                atomicAdd(&s_w2hi[rel], mant >> TT_W2_LOW);
                                atomicAdd(&s_w2lo[rel], (mant & ((1ull << TT_W2_LOW) - 1)) | (1ull << 44));
                            }
                        }
                    }
                    const int bin = e_ - TT_EBASE;
                    const int hd = e_ - hot_lo;
                    if (!direct && ((unsigned)hd < (unsigned)TT_HOT || (unsigned)bin < (unsigned)TT_NB)) {
                        const int f2 = (int)((wb >> 50) & (TT_HSUB - 1));
                        const int slot =
                            (unsigned)hd < (unsigned)TT_HOT ? TT_NB + (hd * TT_HSUB + f2) * TT_HCOPIES + copy : bin;
                        atomicAdd(&s_hi[slot], mant >> 26);
                        atomicAdd(&s_lo[slot], (mant & ((1ull << 26) - 1)) | (1ull << 44));
                    } else {
                        atomicAdd(&b.h1[e_], 1ull);
                        atomicAdd(&b.h1[STS_NBIN + e_], mant >> 26);
                        atomicAdd(&b.h1[2 * STS_NBIN + e_], mant & ((1ull << 26) - 1));
                    }
                }
                c_all += (u32)__popcll(__ballot(cand));
                if (predict) {
                    const u64 m_ab = __ballot(ab), m_in = __ballot(inw);
                    const u32 n_ab = (u32)__popcll(m_ab), n_in = (u32)__popcll(m_in);
                    fits = fits && c_in + c_ab + n_ab + n_in <= room;
                    if (fits) {
                        if (inw) {
                            const u32 at = c_in + sts_lanes_below(m_in);
                            sts_store_at(sk, at * 8u, G.rest | deposit_bits<M>((u32)i, g));
                            sts_store_at(sw, at * 8u, wb);
                            sts_store_at(sa, at * (u32)sizeof(AT), o);
                        } else if (ab) {
                            const u32 at = room - 1u - c_ab - sts_lanes_below(m_ab);
                            sts_store_at(sk, at * 8u, G.rest | deposit_bits<M>((u32)i, g));
                            sts_store_at(sa, at * (u32)sizeof(AT), o);
                        }
                    }
                    c_in += n_in;
                    c_ab += n_ab;
                }
            }
            if (direct && predict) flush_window(s_wacc, ma, mw); // the lane sums are bounded for binned shares only
        });
        if (sts_lane() == 0) {
            b.w_all[sl] = c_all;
            if (predict) {
                b.t_above[sl] = c_ab;
                b.t_side[sl] = c_in;
                if (!fits) atomicOr(&ctl->w_over, 1u);
                atomicAdd((unsigned long long *)&s_wacc[0], (unsigned long long)c_ab);
                atomicAdd((unsigned long long *)&s_wacc[3], (unsigned long long)c_in);
            }
        }
    }
    __syncthreads();
    flush_bins(b, s_hi, s_lo, hot_lo);
    if (fine) flush_w2(b, s_w2hi, s_w2lo, d_lo);
    if (predict) {
        flush_window(s_wacc, ma, mw);
        __syncthreads();
        if (threadIdx.x < 6) b.wpart[threadIdx.x * STS_MAX_GROUPS + blockIdx.x] = s_wacc[threadIdx.x];
    }
}

// ---------------------------------------------------------------------------
// sampling pass (as k_tile_sample): the gate on evenly spaced tiles
// ---------------------------------------------------------------------------
template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_sample(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    __shared__ BktSmem<AT> s;
    __shared__ SampleSmem ss;
    DevCtl *ctl = b.ctl;
    const int e_prev = ctl->e_pred;
    if (e_prev < 0) return; // uniform: nothing to centre the bins on
    clear_slots<AT>(s);
    SampleAcc acc;
    sample_begin(ss);
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
            share_groups<AT, M>(s, g, sh, wv, b.keys, (const AT *)b.amps, [&](const Group<AT, M> &G) {
#pragma unroll
                for (int i = 0; i < (1 << M); ++i) {
                    const AT o = group_out<AT, M>(g, G, i);
                    if (G.present && nonzero(o)) sample_add(ss, acc, weight_bits(o), e_lo);
                }
            });
        }
    }
    sample_flush(ss, acc, b, sts_lane() == 0 ? seen : 0u);
    if (!sts_last_block(&ctl->done[2], &ss.flag)) return;
    sample_finish(ss, b, e_lo, *b.n_in);
}

// ---------------------------------------------------------------------------
// the passes of a step whose window missed the cut (they exit at once when it
// held it): the candidates of the cut's exponent to the side buffer, densely
// packed (one claim per tile), and the survivors per share
// ---------------------------------------------------------------------------
template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_extract(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    __shared__ BktSmem<AT> s;
    __shared__ u32 s_cnt[BW];
    __shared__ u64 s_base;
    DevCtl *ctl = b.ctl;
    if (ctl->pred_hit || ctl->keep_all) return; // uniform
    clear_slots<AT>(s);
    const int e_star = ctl->e_star;
    const u64 *keys = b.keys;
    const AT *amps = (const AT *)b.amps;
    const u32 ntiles = bkt_tiles(g.bkt);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    __syncthreads();
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        u32 cnt = 0;
        share_groups<AT, M>(s, g, sh, wv, keys, amps, [&](const Group<AT, M> &G) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT o = group_out<AT, M>(g, G, i);
                cnt += (u32)__popcll(__ballot(G.present && nonzero(o) && (int)(weight_bits(o) >> 52) == e_star));
            }
        });
        if (sts_lane() == 0) s_cnt[wv] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) s_base = atomicAdd(&ctl->side_n, (u64)s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3]);
        __syncthreads();
        u64 at = s_base;
        for (int w = 0; w < wv; ++w) at += s_cnt[w];
        share_groups<AT, M>(s, g, sh, wv, keys, amps, [&](const Group<AT, M> &G) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT o = group_out<AT, M>(g, G, i);
                const u64 wb = weight_bits(o);
                const bool take = G.present && nonzero(o) && (int)(wb >> 52) == e_star;
                const u64 m = __ballot(take);
                const u64 p = at + sts_lanes_below(m);
                if (take && p < b.side_cap) {
                    b.side_key[p] = G.rest | deposit_bits<M>((u32)i, g);
                    b.side_w[p] = wb;
                }
                at += (u64)__popcll(m);
            }
        });
        __syncthreads();
    }
}

template <typename AT> __device__ __forceinline__ bool survives(u64 wb, u64 key, bool all, u64 thr_w, u64 thr_k)
{
    return all || wb > thr_w || (wb == thr_w && key <= thr_k);
}

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_count(const GateArg *__restrict__ gp, PassBufs b)
{
    const GateArg &g = *gp;
    __shared__ BktSmem<AT> s;
    DevCtl *ctl = b.ctl;
    const bool all = b.materialise;
    if (!all && (ctl->pred_hit || ctl->keep_all)) return; // uniform
    clear_slots<AT>(s);
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const u32 ntiles = bkt_tiles(g.bkt);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    __syncthreads();
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Share sh = load_share(g.bkt, b.bd_in, tile, wv);
        u32 cnt = 0;
        share_groups<AT, M>(s, g, sh, wv, b.keys, (const AT *)b.amps, [&](const Group<AT, M> &G) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT o = group_out<AT, M>(g, G, i);
                const u64 key = G.rest | deposit_bits<M>((u32)i, g);
                cnt += (u32)__popcll(
                    __ballot(G.present && nonzero(o) && survives<AT>(weight_bits(o), key, all, thr_w, thr_k)));
            }
        });
        if (sts_lane() == 0) b.w_kept[(tile << 2) + (u32)wv] = cnt;
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
    u64 peers = __ballot(keep);
    for (int t = 0; t < bits; ++t) {
        const u64 bb = __ballot((sub >> t) & 1u);
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

template <typename AT, int M>
__global__ void __launch_bounds__(STS_WG) k_bkt_emit(const GateArg *__restrict__ gp, PassBufs b)
{
    constexpr int UN = 8; // items of a share held in registers
    const GateArg &g = *gp;
    __shared__ BktSmem<AT> s;
    __shared__ u32 s_cnt[BW][BW_SUBS];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const u32 lane = (u32)sts_lane();
    const u32 tile = blockIdx.x;
    const DevCtl *ctl = b.ctl;
    const int keep_all = ctl->keep_all, dropped = ctl->dropped, hit = ctl->pred_hit;
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const double scale = ctl->scale;
    const bool all = b.materialise || keep_all;
    const bool rescale = !all && dropped;
    const BktPlan &p = g.bkt;
    const int bits = 2 + p.delta;
    const u32 sl = (tile << 2) + (u32)wv;
    u32 *cnt = s_cnt[wv];
    cnt[lane] = 0;
    u64 base64 = b.t_off[tile];
    for (int w = 0; w < wv; ++w) base64 += b.w_kept[(tile << 2) + (u32)w];
    const u32 base = (u32)base64;
    wave_sync();
    const u32 cap = (u32)b.out_cap;
    u64 *ok = b.out_keys;
    AT *oa = (AT *)b.out_amps;
    if (!all && hit) {
        const int shift = ctl->side_slab_shift;
        const u32 na = b.t_above[sl], ns = b.t_side[sl], n = na + ns;
        const u64 slab = (u64)sl << shift;
        const u64 ab0 = slab + (1ull << shift) - na; // the entries above the window
        const AT *sa = (const AT *)b.side_amp;
        auto place = [&](u32 j) { return j < na ? ab0 + j : slab + (j - na); };
        if (n <= UN * 64) {
            u64 kk[UN];
            AT aa[UN];
            u64 ww[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = (u32)r * 64 + lane;
                ww[r] = 0;
                if (j < n) {
                    const u64 i = place(j);
                    kk[r] = __builtin_nontemporal_load(&b.side_key[i]);
                    aa[r].x = __builtin_nontemporal_load(&sa[i].x);
                    aa[r].y = __builtin_nontemporal_load(&sa[i].y);
                    if (j >= na) ww[r] = b.side_w[i];
                }
            }
            u32 pos[UN], sub[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = (u32)r * 64 + lane;
                const bool keep = j < n && (j < na || survives<AT>(ww[r], kk[r], false, thr_w, thr_k));
                sub[r] = keep ? sub_bucket(p, kk[r]) : 0u;
                pos[r] = sub_rank(keep, sub[r], bits, cnt);
                if (!keep) sub[r] = ~0u;
            }
            wave_sync();
            sub_starts(p, b, tile, wv, base, cnt);
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                if (sub[r] == ~0u) continue;
                const u32 at = cnt[sub[r]] + pos[r];
                if (at < cap) {
                    ok[at] = kk[r];
                    const AT o = out_amp(aa[r], rescale, scale);
                    __builtin_nontemporal_store(o.x, &oa[at].x);
                    __builtin_nontemporal_store(o.y, &oa[at].y);
                }
            }
            return;
        }
        // a large share: count, then place
        for (int phase = 0; phase < 2; ++phase) {
            for (u32 j0 = 0; j0 < n; j0 += 64) {
                const u32 j = j0 + lane;
                bool keep = false;
                u64 k = 0, i = 0;
                if (j < n) {
                    i = place(j);
                    k = b.side_key[i];
                    keep = j < na || survives<AT>(b.side_w[i], k, false, thr_w, thr_k);
                }
                const u32 at = sub_rank(keep, keep ? sub_bucket(p, k) : 0u, bits, cnt);
                if (phase && keep && at < cap) {
                    ok[at] = k;
                    oa[at] = out_amp(sa[i], rescale, scale);
                }
            }
            wave_sync();
            if (phase == 0) sub_starts(p, b, tile, wv, base, cnt);
        }
        return;
    }
    // recompute
    clear_slots<AT>(s);
    __syncthreads();
    const Share sh = load_share(p, b.bd_in, tile, wv);
#pragma unroll 1
    for (int phase = 0; phase < 2; ++phase) {
        share_groups<AT, M>(s, g, sh, wv, b.keys, (const AT *)b.amps, [&](const Group<AT, M> &G) {
#pragma unroll
            for (int i = 0; i < (1 << M); ++i) {
                const AT o = group_out<AT, M>(g, G, i);
                const u64 key = G.rest | deposit_bits<M>((u32)i, g);
                const bool keep =
                    G.present && nonzero(o) && survives<AT>(weight_bits(o), key, all, thr_w, thr_k);
                const u32 at = sub_rank(keep, keep ? sub_bucket(p, key) : 0u, bits, cnt);
                if (phase && keep && at < cap) {
                    ok[at] = key;
                    oa[at] = out_amp(o, rescale, scale);
                }
            }
        });
        if (phase == 0) sub_starts(p, b, tile, wv, base, cnt);
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
template <typename AT, int M> int hist_capacity_b()
{
    static const int cap = [] {
        int per_cu = 0, dev = 0, cus = 0;
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_bkt_hist<AT, M>, STS_WG, 0);
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        return std::min((per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1), STS_MAX_GROUPS);
    }();
    return cap;
}

template <typename AT, int M> hipError_t launch_m(int kind, const PassBufs &b, int tiles, hipStream_t s)
{
    const int cap = hist_capacity_b<AT, M>();
    switch (kind) {
    case STS_BKT_HIST:
        hipLaunchKernelGGL((k_bkt_hist<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_SAMPLE:
        hipLaunchKernelGGL((k_bkt_sample<AT, M>), dim3(STS_SAMPLE_TILES / 2), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_EXTRACT:
        hipLaunchKernelGGL((k_bkt_extract<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_COUNT:
        hipLaunchKernelGGL((k_bkt_count<AT, M>), dim3(std::min(tiles, cap)), dim3(STS_WG), 0, s, b.gate, b);
        break;
    case STS_BKT_EMIT:
        hipLaunchKernelGGL((k_bkt_emit<AT, M>), dim3(tiles), dim3(STS_WG), 0, s, b.gate, b);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

} // namespace sts_bucket
