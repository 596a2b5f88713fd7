// select.hip - finding the cut of a truncation exactly.
//
// Truncation keeps the shortest prefix of the terms ranked by (|a|^2
// descending, key ascending) that holds at least p of the mass, and at most K
// terms (Sec. III; the ranking by decreasing |a|^2 of Sec. IV.B). Instead of
// sorting all candidates, the cut is located by most-significant-digit
// selection on the rank:
//   level 1  - the exponent field of |a|^2 (2048 bins, from the histogram
//              pass over the recomputed candidates),
//   level 2  - within that exponent, the top 11 bits of the within-exponent
//              rank key V = ((2^52 - 1 - fraction) << 64) | key, from the side
//              buffer of that exponent's candidates,
//   level 3+ - further 11-bit digits of V inside one workgroup (level 3 from
//              a histogram built while the level-2 subset is copied out),
//              until at most 128 terms remain, whose ranks are counted.
// Masses are exact: each bin carries the exact integer sum of its weights'
// mantissas, levels >= 2 share one exponent, and level 1 prefixes are exact
// integers on the 2^-1074 grid. Every decision therefore equals the one made
// in exact arithmetic, and the kept mass S is correctly rounded.
#include <algorithm>

#include "kernels.h"
#include "select_impl.h"

namespace {

using namespace sts_select;

__global__ void __launch_bounds__(256) k_pick1(PassBufs b, int groups, int peak_only, int predicted)
{
    __shared__ Level1Smem<256> sm;
    pick_level1<256>(b, groups, peak_only, predicted, sm, DeviceBins<256>{b.h1});
}

// ---------------------------------------------------------------------------
// level 1 and 2 of a sampled bucketed step, from the weighing pass's sums:
// the exact total W, the exact mass above the window, and the window's level-2
// bins. Decides exactly whether the window holds the cut; if so picks level 2,
// if nothing is cut says so, and otherwise asks for the histogram pass.
// A chain of latencies: 12 us at 2^20 complex128 terms, 16 at 2^24 complex64
// ones; limbs and carries of the exponent bins are added apart (12.9 and 17 us with a
// carry resolved for every bin).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_pick_window(PassBufs b, int groups)
{
    __shared__ unsigned short s_e[STS_NBIN]; // the non-empty exponent bins in rank order
    __shared__ __attribute__((aligned(16))) u64 s_p[3][STS_NBIN]; // their mantissa sums, as the limbs from (unit bit / 64) on
    __shared__ u32 s_scan[4];
    __shared__ u64 s_cnt[4][3];
    __shared__ u64 s_sum[4][6]; // per wave: total, above, window (low and high words)
    __shared__ u64 s_part[4][2][64];
    __shared__ Sub s_sub;
    __shared__ u32 s_fine, s_hit2;
    __shared__ u64 s_R_lo, s_R_hi;
    const int t = threadIdx.x, lane = t & 63, q = t >> 6;
    DevCtl *ctl = b.ctl;
    u64 *h1 = b.h1;
    const int w_mode = ctl->w_mode, e = ctl->e_w;
    const u32 over = ctl->w_over;
    const u64 w_hi = ctl->w_hi;
    if (t == 0) {
        s_fine = 0;
        ctl->slab_all = 0;
    }
    __syncthreads(); // the control words are read
    if (!w_mode || over) { // uniform: the histogram pass has to do the step
        if (t == 0) {
            ctl->need_full = 1;
            ctl->w_mode = 0;
            ctl->w_over = 0;
            ctl->w2_mode = 0;
            ctl->l2_done = 0;
        }
        if (w_mode)
            for (int i = t; i < 3 * STS_NBIN; i += 256) {
                h1[i] = 0;
                st_agent(&b.h2w[i], 0ull);
            }
        return;
    }
    const int L = ctl->w_L;
    // every load issued before any is used: the workgroups' sums,
    u64 c_all = 0, c_ab = 0, c_in = 0;
    u128 tot = 0, abv = 0; // units of 2^(L - 1075); the low parts may be negative
#pragma unroll
    for (int r = 0; r < STS_MAX_GROUPS / 256; ++r) {
        const int i = t + 256 * r;
        if (i < groups) {
            const u64 *w = b.wpart + i;
            tot += ((u128)w[0] << 40) + (u128)(__int128)(long long)w[STS_MAX_GROUPS];
            abv += ((u128)w[2 * STS_MAX_GROUPS] << 40) + (u128)(__int128)(long long)w[3 * STS_MAX_GROUPS];
            c_all += w[4 * STS_MAX_GROUPS];
            c_ab += w[5 * STS_MAX_GROUPS];
            c_in += w[6 * STS_MAX_GROUPS];
        }
    }
    // the window's level-2 bins,
    const u32 d_lo = (u32)((((1ull << 52) - 1) - (w_hi & ((1ull << 52) - 1))) >> 41);
    u128 win = 0;
    if (t < 192 && d_lo + (u32)t < STS_NBIN)
        win = ((u128)ld_agent(&b.h2w[STS_NBIN + d_lo + t]) << 26) + (u128)ld_agent(&b.h2w[2 * STS_NBIN + d_lo + t]);
    // and the exponent bins (weights far from the window)
    u64 c[8], hi[8], lo[8];
    u32 nz = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int f = 2047 - 8 * t - k;
        c[k] = h1[f];
        hi[k] = h1[STS_NBIN + f];
        lo[k] = h1[2 * STS_NBIN + f];
        nz += c[k] ? 1u : 0u;
    }
    u32 nbins;
    u32 at = block_excl_scan<u32, 256>(nz, s_scan, &nbins);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (!c[k]) continue;
        s_e[at] = (unsigned short)(2047 - 8 * t - k);
        const u128 ms = ((u128)hi[k] << 26) + (u128)lo[k];
        const int off = unit_bit(2047 - 8 * t - k) & 63;
        const u128 ml = ms << off;
        s_p[0][at] = (u64)ml;
        s_p[1][at] = (u64)(ml >> 64);
        s_p[2][at] = off ? (u64)(ms >> 64) >> (64 - off) : 0ull;
        ++at;
    }
    tot = wave_incl_scan(tot); // (lane 63: the sum)
    abv = wave_incl_scan(abv);
    win = wave_incl_scan(win);
    c_all = wave_incl_scan(c_all);
    c_ab = wave_incl_scan(c_ab);
    c_in = wave_incl_scan(c_in);
    if (lane == 63) {
        s_cnt[q][0] = c_all;
        s_cnt[q][1] = c_ab;
        s_cnt[q][2] = c_in;
        const u128 v[3] = {tot, abv, win};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            s_sum[q][2 * i] = (u64)v[i];
            s_sum[q][2 * i + 1] = (u64)(v[i] >> 64);
        }
    }
    __syncthreads();
    {
        // the exponent bins in four chunks, one wave each: those above the
        // register range, then those below
        const u32 chunk = (nbins + 3) / 4;
        const u32 j0 = (u32)q * chunk, j1 = j0 + chunk < nbins ? j0 + chunk : nbins;
        // limbs and their carries apart; the carries are resolved at the end
        u64 A = 0, B = 0;
        u32 cA = 0, cB = 0;
#pragma unroll 4
        for (u32 j = j0; j < j1; ++j) {
            const int f = (int)s_e[j];
            const u32 k = (u32)lane - ((u32)unit_bit(f) >> 6);
            const u64 v = k < 3u ? s_p[k][j] : 0ull;
            if (f >= L) { // uniform
                A += v;
                cA += A < v ? 1u : 0u;
            } else {
                B += v;
                cB += B < v ? 1u : 0u;
            }
        }
        const u32 upA = __shfl_up(cA, 1, 64), upB = __shfl_up(cB, 1, 64);
        A = wl_add(A, lane ? (u64)upA : 0ull);
        B = wl_add(B, lane ? (u64)upB : 0ull);
        s_part[q][0][lane] = A;
        s_part[q][1][lane] = B;
    }
    __syncthreads();
    if (t < 64) { // one wave decides
        u64 Sa = 0, W = 0;
        c_all = c_ab = c_in = 0;
        tot = abv = win = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            Sa = wl_add(Sa, s_part[i][0][lane]);
            W = wl_add(W, s_part[i][1][lane]);
            c_all += s_cnt[i][0];
            c_ab += s_cnt[i][1];
            c_in += s_cnt[i][2];
            tot += make128(s_sum[i][0], s_sum[i][1]);
            abv += make128(s_sum[i][2], s_sum[i][3]);
            win += make128(s_sum[i][4], s_sum[i][5]);
        }
        W = wl_add(wl_add(W, Sa), wl_piece((u64)tot, (u64)(tot >> 64), unit_bit(L)));
        Sa = wl_add(Sa, wl_piece((u64)abv, (u64)(abv >> 64), unit_bit(L)));
        const u64 K = ctl->K;
        const double p = ctl->p;
        const bool p_on = p > 0.0 && p < 1.0;
        u64 T = 0; // p-mass target ceil(p * W), exactly
        if (p_on) {
            const u64 pb = sts_dbits(p);
            const u64 pe = pb >> 52, pf = pb & ((1ull << 52) - 1);
            T = wl_mul_shr_ceil(W, pe ? (pf | (1ull << 52)) : pf, pe ? (int)(1075 - pe) : 1074);
        }
        const bool met_all = (K > 0 && c_all >= K) || (p_on && wl_cmp(W, T) >= 0);
        const bool met_a = (K > 0 && c_ab >= K) || (p_on && wl_cmp(Sa, T) >= 0);
        const u64 Sw = wl_add(Sa, wl_piece((u64)win, (u64)(win >> 64), unit_bit(e)));
        const bool met_w = (K > 0 && c_ab + c_in >= K) || (p_on && wl_cmp(Sw, T) >= 0);
        const bool hit = !met_a && met_w;
        const double Wd = wl_to_double(W);
        u64 R_lo = ~0ull, R_hi = ~0ull; // mass still to reach inside the window, in its units (rounded up)
        if (p_on && hit) {
            bool sticky;
            const u64 r0 = wl_shr(wl_sub(T, Sa), unit_bit(e), &sticky);
            const bool big = __ballot(lane >= 2 && r0 != 0) != 0;
            u128 r = ((u128)__shfl(r0, 1, 64) << 64) | (u128)__shfl(r0, 0, 64);
            if (!big) {
                if (sticky) r += 1;
                if (r != 0 || !sticky) {
                    R_lo = (u64)r;
                    R_hi = (u64)(r >> 64);
                }
            }
        }
        if (hit && lane < STS_NL) ctl->S_excl.l[lane] = Sa;
        if (lane < STS_NL) ctl->T.l[lane] = T;
        if (lane == 0) {
            ctl->w_mode = 0;
            ctl->w2_mode = 0;
            ctl->l2_done = 0;
            if (met_all && !hit) {
                ctl->need_full = 1; // the cut lies elsewhere
            } else {
                ctl->cand_all = c_all;
                ctl->W = Wd;
                ctl->n_cand = c_all;
                ctl->tot_steps += 1;
                ctl->tot_updates += *b.n_in;
                ctl->tot_cand += c_all;
                ctl->level = 1;
                if (!met_all) {
                    ctl->keep_all = 1;
                    ctl->dropped = 0;
                    ctl->L = c_all;
                    ctl->scale = 1.0;
                    ctl->S = Wd;
                    ctl->frac = 1.0;
                    ctl->pred_hit = 0;
                    ctl->e_pred = -1;
                } else {
                    ctl->keep_all = 0;
                    ctl->pred_hit = 1;
                    ctl->e_pred = e;
                    ctl->e_star = e;
                    ctl->R_lo = R_lo;
                    ctl->R_hi = R_hi;
                    s_fine = 1;
                    s_sub.cnt_before = c_ab;
                    s_sub.mb = 0; // S_excl holds all the mass above the window
                    s_sub.vpre = 0;
                    s_sub.vshift = 116;
                    s_sub.count = c_in;
                    s_R_lo = R_lo;
                    s_R_hi = R_hi;
                }
            }
        }
    }
    __syncthreads();
    if (nbins)
        for (int i = t; i < 3 * STS_NBIN; i += 256) h1[i] = 0;
    if (s_fine) { // uniform: the bin lists above are done with, so their LDS serves the pick
        const bool ok = pick_digit<256>(AgentBins{b.h2w}, ctl->K,
                                        make128(s_R_lo, s_R_hi), 11, &s_sub, reinterpret_cast<u128 *>(s_p[0]), s_p[1],
                                        &s_hit2);
        if (ok && t <= STS_SUB_REGIONS) st_agent(&b.sub_cnt[t * 32], 0u);
        if (t == 0) {
            if (ok) {
                sub_store(s_sub, ctl);
                ctl->level = 2;
                ctl->l2_done = 1;
            } else {
                atomicOr(&ctl->flags, STS_F_UNRESOLVED);
            }
        }
    }
    __syncthreads();
    if (t < 192 && d_lo + (u32)t < STS_NBIN) {
#pragma unroll
        for (int f = 0; f < 3; ++f) st_agent(&b.h2w[f * STS_NBIN + d_lo + t], 0ull);
    }
}

// The side buffer is either dense (entries [0, side_n)) or split into slabs
// of 2^shift entries (one per tile, or one per wave of a tile in the
// histogram pass), slab s holding t_side[s] entries from its start. Its
// entries are visited through a flat index f over the whole layout.
struct SideView {
    const u64 *key;
    const u64 *w;
    const u32 *cnt;
    u64 flat;  // flat indices to visit
    int dense;
    int shift;
};

__device__ __forceinline__ SideView side_view(const PassBufs &b, const DevCtl *ctl)
{
    SideView v;
    v.key = b.side_key;
    v.w = b.side_w;
    v.cnt = b.t_side;
    v.dense = ctl->side_dense;
    v.shift = ctl->side_slab_shift;
    const u64 f = v.dense ? ctl->side_n : (ctl->side_ntiles << v.shift);
    v.flat = f < b.side_cap ? f : b.side_cap;
    return v;
}

// The same entries as a list of chunks: the tiles of the tiled layout (each
// the runs of its 1 or 4 slabs), or runs of 8192 entries of the dense one.
// Workgroups walk chunks; threads walk the entries of a chunk.
struct SideChunks {
    u64 nchunks;
    int dense;
    int shift;
    int spl;
    u64 n;          // dense: entries
    u64 cap;
    const u32 *cnt;
};

__device__ __forceinline__ SideChunks side_chunks(const PassBufs &b, const DevCtl *ctl)
{
    SideChunks c;
    c.dense = ctl->side_dense;
    c.shift = ctl->side_slab_shift;
    c.spl = ctl->side_spt_log2;
    c.cap = b.side_cap;
    c.cnt = b.t_side;
    c.n = ctl->side_n < b.side_cap ? ctl->side_n : b.side_cap;
    c.nchunks = c.dense ? (c.n + 8191) / 8192 : (ctl->side_ntiles >> c.spl);
    return c;
}

// the entries of chunk t (visited with slab_at)
__device__ __forceinline__ TileSlabs chunk_of(const SideChunks &c, u64 t)
{
    if (!c.dense) return tile_slabs(c.cnt, t, c.spl, c.shift, false, c.cap);
    TileSlabs s;
    const u64 base = t * 8192;
    const u32 count = (u32)(c.n - base < 8192 ? c.n - base : 8192);
    s.f0 = base;
    s.f1 = s.f2 = s.f3 = 0;
    s.p1 = s.p2 = s.p3 = s.n = count;
    return s;
}

// most entries a chunk can hold
__device__ __forceinline__ u64 chunk_max(const SideChunks &c) { return c.dense ? 8192ull : (1ull << (c.shift + c.spl)); }

// ---------------------------------------------------------------------------
// level 2 over the side buffer (many workgroups), pick by the last one
// ---------------------------------------------------------------------------
// LDS bins of the level-2 histogram: s_hi sums mantissa >> 20, s_lo sums
// mantissa & (2^20 - 1) plus count << 44. A workgroup flushes them before
// 2^19 entries have gone in, so neither field can overflow into the next.
constexpr int SH_LOW = 20;
constexpr u64 SH_FLUSH = 1ull << 19;

__device__ __forceinline__ void side_flush(u64 *h2, u64 *s_hi, u64 *s_lo)
{
    for (int i = threadIdx.x; i < STS_NBIN; i += 256) {
        const u64 lo = s_lo[i];
        const u64 c = lo >> 44;
        if (c) {
            const u128 tot = ((u128)s_hi[i] << SH_LOW) + (u128)(lo & ((1ull << 44) - 1));
            atomicAdd(&h2[i], c);
            atomicAdd(&h2[STS_NBIN + i], (u64)(tot >> 26));
            atomicAdd(&h2[2 * STS_NBIN + i], (u64)tot & ((1ull << 26) - 1));
        }
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
}

// this workgroup's share of the level-2 histogram of the side buffer, added
// to h2
__device__ __forceinline__ void side_bins(const PassBufs &b, DevCtl *ctl, u64 *h2, u64 *s_hi, u64 *s_lo)
{
    constexpr int UN = 16; // entries in flight per lane
    for (int i = threadIdx.x; i < STS_NBIN; i += 256) {
        s_hi[i] = 0;
        s_lo[i] = 0;
    }
    __syncthreads();
    const SideChunks sc = side_chunks(b, ctl);
    // each wave takes a chunk of its own, so a workgroup has four chunks'
    // loads in flight; a round of four chunks adds at most 4 * chunk_max
    // entries, and the bins are flushed before they could overflow
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const u64 cmax = chunk_max(sc);
    u64 since = 0;
    for (u64 r0 = (u64)blockIdx.x * 4; r0 < sc.nchunks; r0 += (u64)gridDim.x * 4) {
        if (since + 4 * cmax > SH_FLUSH) { // uniform across the workgroup
            __syncthreads();
            side_flush(h2, s_hi, s_lo);
            __syncthreads();
            since = 0;
        }
        since += 4 * cmax;
        const u64 t = r0 + wv;
        if (t >= sc.nchunks) continue;
        const TileSlabs ch = chunk_of(sc, t);
        const u32 count = ch.n;
        for (u32 i0 = 0; i0 < count; i0 += UN * 64) {
            u64 w[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 i = i0 + (u32)r * 64 + lane;
                w[r] = i < count ? b.side_w[slab_at(ch, i)] : ~0ull;
            }
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                if (w[r] == ~0ull) continue; // past the chunk (no weight has all bits set)
                const u64 vh = ((1ull << 52) - 1) - (w[r] & ((1ull << 52) - 1));
                const u32 d = (u32)(vh >> 41);
                const u64 mant = sts_mant(w[r]);
                atomicAdd(&s_hi[d], mant >> SH_LOW);
                atomicAdd(&s_lo[d], (mant & ((1ull << SH_LOW) - 1)) | (1ull << 44));
            }
        }
    }
    __syncthreads();
    side_flush(h2, s_hi, s_lo);
}

__global__ void __launch_bounds__(256) k_side_hist(PassBufs b, u64 *h2)
{
    __shared__ u64 s_hi[STS_NBIN];
    __shared__ u64 s_lo[STS_NBIN];
    __shared__ u128 s_m[4]; // a wave's each
    __shared__ u64 s_c[4];
    __shared__ u32 s_hit, s_flag;
    __shared__ Sub s_sub;
    DevCtl *ctl = b.ctl;
    const int keep_all = ctl->keep_all, w2 = ctl->w2_mode;
    // the level-1 pick already picked level 2 from the histogram pass's
    // window bins
    if (ctl->l2_done) return;
    // the histogram pass binned a sampled window that holds the cut: its
    // level-2 bins are complete, and only the pick is left
    const bool fine = w2 && ctl->pred_hit && !keep_all;
    if (keep_all && !w2) return;
    if (!keep_all && !fine) side_bins(b, ctl, h2, s_hi, s_lo);
    if (!sts_last_block(&ctl->done[1], &s_flag)) return;
    if (!keep_all) {
        const u64 *hs = fine ? b.h2w : h2;
        if (threadIdx.x == 0) {
            s_sub.cnt_before = ctl->cnt_before;
            s_sub.mb = make128(ctl->mb_lo, ctl->mb_hi); // the window's exponent above it, or 0
            s_sub.vpre = 0;
            s_sub.vshift = 116;
            s_sub.count = ctl->sub_count;
        }
        __syncthreads();
        const u128 R = make128(ctl->R_lo, ctl->R_hi);
        if (pick_digit<256>(AgentBins{hs}, ctl->K, R, 11, &s_sub, s_m, s_c, &s_hit)) {
            if (threadIdx.x <= STS_SUB_REGIONS) st_agent(&b.sub_cnt[threadIdx.x * 32], 0u);
            if (threadIdx.x == 0) {
                sub_store(s_sub, ctl);
                ctl->level = 2;
            }
        } else if (threadIdx.x == 0) {
            atomicOr(&ctl->flags, STS_F_UNRESOLVED);
        }
        if (!fine)
            for (int i = threadIdx.x; i < 3 * STS_NBIN; i += 256) st_agent(&h2[i], 0ull);
    }
    if (w2)
        for (int i = threadIdx.x; i < 3 * STS_NBIN; i += 256) st_agent(&b.h2w[i], 0ull);
}


// ---------------------------------------------------------------------------
// copy the level-2 subset out of the side buffer (many workgroups), so the
// final workgroup reads a few thousand terms instead of the whole buffer
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_side_extract(PassBufs b)
{
    constexpr int UN = 4;
    DevCtl *ctl = b.ctl;
    // every control load issued before any is used
    const int keep_all = ctl->keep_all;
    const u32 flags = ctl->flags;
    const u64 sub_count = ctl->sub_count;
    const SideChunks sc = side_chunks(b, ctl);
    const int vshift = ctl->vshift;
    const u128 vpre = make128(ctl->vpre_lo, ctl->vpre_hi);
    const int e = ctl->e_star;
    if (keep_all || (flags & (STS_F_UNRESOLVED | STS_F_SIDE_OVERFLOW))) return;
    if (sub_count > b.sub_cap) return; // the final kernel reads the side buffer itself
    // the subset's histogram for the next level (the digit below vshift),
    // with exact mantissa sums, as the final workgroup's first level would
    // bin it: that workgroup then starts from the pick
    const int dw = vshift < 11 ? vshift : 11;
    // each wave fills one of STS_SUB_REGIONS regions, whose counters sit on
    // separate cache lines (one shared counter would serialise every wave)
    const u32 region = (blockIdx.x * 4u + (threadIdx.x >> 6)) % STS_SUB_REGIONS;
    const u32 region_len = (u32)(b.sub_cap / STS_SUB_REGIONS);
    const u64 region_base = (u64)region * region_len;
    u32 *cnt = &b.sub_cnt[region * 32];
    const u64 lt = sts_lanemask_lt();
    // tiles (a few hundred window entries each): one wave per tile, so that
    // every tile's wave is resident at once; dense runs: a workgroup per run
    const bool per_wave = !sc.dense;
    const u32 wv = threadIdx.x >> 6;
    const u64 t0 = per_wave ? (u64)blockIdx.x * 4 + wv : (u64)blockIdx.x;
    const u64 tstep = per_wave ? (u64)gridDim.x * 4 : (u64)gridDim.x;
    const u32 nth = per_wave ? 64u : 256u, me = per_wave ? (u32)sts_lane() : (u32)threadIdx.x;
    for (u64 t = t0; t < sc.nchunks; t += tstep) {
        const TileSlabs ch = chunk_of(sc, t);
        const u32 count = ch.n;
        for (u32 i0 = 0; i0 < count; i0 += UN * nth) {
            u64 w[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = i0 + (u32)r * nth + me;
                w[r] = j < count ? b.side_w[slab_at(ch, j)] : ~0ull;
            }
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 j = i0 + (u32)r * nth + me;
                const u64 i = j < count ? slab_at(ch, j) : 0ull;
                bool take = false;
                u64 k = 0;
                if (w[r] != ~0ull) {
                    if (vshift >= 64) { // the fixed part lies in the weight half of V
                        const u64 vh = ((1ull << 52) - 1) - (w[r] & ((1ull << 52) - 1));
                        take = (int)(w[r] >> 52) == e && (vh >> (vshift - 64)) == (u64)vpre;
                        if (take) k = b.side_key[i];
                    } else {
                        k = b.side_key[i];
                        take = (int)(w[r] >> 52) == e && (rank_key(w[r], k) >> vshift) == vpre;
                    }
                }
                const u64 mask = __ballot(take);
                if (!mask) continue;
                const int leader = __ffsll((long long)mask) - 1;
                u32 pos = 0;
                if (sts_lane() == leader) {
                    pos = atomicAdd(cnt, (u32)__popcll(mask));
                    if (pos + (u32)__popcll(mask) > region_len) atomicOr(&b.sub_cnt[STS_SUB_REGIONS * 32], 1u);
                }
                pos = __shfl(pos, leader, 64) + (u32)__popcll(mask & lt);
                if (take && pos < region_len) {
                    b.sub_key[region_base + pos] = k;
                    b.sub_w[region_base + pos] = w[r];
                }
                if (take && dw > 0) {
                    const u128 v = rank_key(w[r], k);
                    const u32 d = (u32)((v >> (vshift - dw)) & (u128)((1u << dw) - 1));
                    const u64 mant = mant_of_v(v, e);
                    atomicAdd(&b.h3[d], 1ull);
                    atomicAdd(&b.h3[STS_NBIN + d], mant >> 26);
                    atomicAdd(&b.h3[2 * STS_NBIN + d], mant & ((1ull << 26) - 1));
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// final levels and the exact cut, one workgroup of 1024 threads
// ---------------------------------------------------------------------------
constexpr int FT = 1024;
constexpr int FB = 8; // subset entries a thread of the final workgroup loads at a time

__global__ void __launch_bounds__(FT) k_final(PassBufs b)
{
    // LDS: the level histograms and the last terms share one region
    __shared__ __attribute__((aligned(16))) unsigned char s_raw[3 * STS_NBIN * sizeof(u64)];
    __shared__ CutSmem s_cut;

    __shared__ Sub s_sub;
    DevCtl *ctl = b.ctl;
    if (ctl->keep_all) return;
    if (ctl->flags & (STS_F_UNRESOLVED | STS_F_SIDE_OVERFLOW)) return;
    const int t = threadIdx.x;
    const int e = ctl->e_star;
    // the subset and what the cut's thread needs at the end, loaded now
    // (visible after the barrier below)
    __shared__ u64 s_Sx[STS_NL], s_ncand;
    __shared__ double s_W, s_l10;
    if (t == 0) {
        sub_load(s_sub, ctl);
        s_ncand = ctl->n_cand;
        s_W = ctl->W;
        s_l10 = ctl->log10_cum;
    }
    if (t < STS_NL) s_Sx[t] = ctl->S_excl.l[t];
    // the subset regions when they hold the whole subset, else the side buffer
    // (entries of region r at r * region_len + [0, count_r); visited through
    // an exclusive prefix of the counts, so only filled slots are read)
    __shared__ u32 s_regpre[STS_SUB_REGIONS + 1];
    const u32 region_len = (u32)(b.sub_cap / STS_SUB_REGIONS);
    const bool small = ctl->sub_count <= b.sub_cap && ld_agent(&b.sub_cnt[STS_SUB_REGIONS * 32]) == 0u;
    if (t < 64) { // one wave scans the region counts
        static_assert(STS_SUB_REGIONS == 64, "one lane per region");
        const u32 c0 = ld_agent(&b.sub_cnt[t * 32]);
        const u32 c = c0 < region_len ? c0 : region_len;
        const u32 inc = (u32)wave_incl_scan((u64)c);
        s_regpre[t + 1] = inc;
        if (t == 0) s_regpre[0] = 0;
    }
    __syncthreads();
    const u64 *src_w = small ? b.sub_w : b.side_w;
    const u64 *src_k = small ? b.sub_key : b.side_key;
    const SideView view = side_view(b, ctl);
    const bool slabs = !small && !view.dense;
    const u64 n = small ? (u64)s_regpre[STS_SUB_REGIONS] : view.flat;
    // physical index of visited entry f of the regions
    auto entry = [&](u64 f) -> u64 {
        if (!small) return f;
        int lo = 0; // the last region r with pre[r] <= f (then f < pre[r + 1])
#pragma unroll
        for (int step = STS_SUB_REGIONS / 2; step > 0; step >>= 1)
            if (s_regpre[lo + step] <= f) lo += step;
        return (u64)lo * region_len + (f - s_regpre[lo]);
    };
    // body(V) for every visited entry whose V lies under the prefix: FB
    // entries per thread at a time, their loads in flight together (a loop
    // of one entry at a time waits on a load per entry)
    auto each_in_subset = [&](int vshift, u128 vpre, bool, auto body) {
        auto take = [&](u64 w, u64 k) {
            const u128 v = rank_key(w, k);
            if ((int)(w >> 52) == e && (v >> vshift) == vpre) body(v);
        };
        if (slabs) { // a wave's slabs, the counts of 64 of them read together
            const u64 room = 1ull << view.shift, nsl = (view.flat + room - 1) >> view.shift;
            for (u64 s0 = (u64)(t >> 6) * 64; s0 < nsl; s0 += FT) {
                const u64 sl = s0 + (u64)sts_lane();
                u64 ns = sl < nsl ? std::min((u64)view.cnt[sl], room) : 0ull;
                if (sl < nsl) ns = std::min(ns, view.flat - (sl << view.shift));
                if (!__ballot(ns != 0)) continue;
#pragma unroll 1
                for (int j = 0; j < 64; j += FB) { // FB slabs at a time
                    u32 nr[FB], most = 0;
#pragma unroll
                    for (int r = 0; r < FB; ++r) {
                        nr[r] = sts_readlane((u32)ns, j + r);
                        most = nr[r] > most ? nr[r] : most;
                    }
                    for (u32 i = (u32)sts_lane(); i < most; i += 64) {
                        u64 w[FB], k[FB];
#pragma unroll
                        for (int r = 0; r < FB; ++r) {
                            const u64 at = i < nr[r] ? ((s0 + (u64)(j + r)) << view.shift) + i : 0ull; // (or a harmless load)
                            w[r] = src_w[at];
                            k[r] = src_k[at];
                        }
#pragma unroll
                        for (int r = 0; r < FB; ++r)
                            if (i < nr[r]) take(w[r], k[r]);
                    }
                }
            }
            return;
        }
        for (u64 f0 = t; f0 < n; f0 += (u64)FT * FB) {
            u64 w[FB], k[FB], at[FB];
            bool ok[FB];
#pragma unroll
            for (int r = 0; r < FB; ++r) {
                const u64 f = f0 + (u64)FT * r;
                ok[r] = f < n;
                at[r] = ok[r] ? entry(f) : 0ull; // entry 0 exists: a harmless load
            }
#pragma unroll
            for (int r = 0; r < FB; ++r) {
                w[r] = src_w[at[r]];
                k[r] = src_k[at[r]];
            }
#pragma unroll
            for (int r = 0; r < FB; ++r)
                if (ok[r]) take(w[r], k[r]);
        }
    };
    const u64 K = ctl->K;
    const u128 R = make128(ctl->R_lo, ctl->R_hi);
    // the subset copy binned the first of the levels below (the condition
    // under which it copies the subset); the bins are cleared here for the
    // next step, whether or not a level is needed
    bool from_h3 = ctl->sub_count <= b.sub_cap;

    // the first level's pick from those bins, then the levels and the cut
    bool ok = true;
    if (from_h3 && s_sub.count > STS_FINAL_SORT && s_sub.vshift > 0)
        ok = pick_digit<FT>(AgentBins{b.h3}, K, R,
                            s_sub.vshift < 11 ? s_sub.vshift : 11, &s_sub, s_cut.m, s_cut.c, &s_cut.hit);
    if (from_h3)
        for (int i = t; i < 3 * STS_NBIN; i += FT) st_agent(&b.h3[i], 0ull);
    ok = ok && resolve_cut<FT, false>(each_in_subset, e, K, R, s_sub, s_raw, s_cut);
    if (!ok) {
        if (t == 0) atomicOr(&ctl->flags, STS_F_UNRESOLVED);
        return;
    }
    if (t < 64) finish_cut(ctl, s_cut, e, s_Sx, s_ncand, s_W, s_l10);
}

// ---------------------------------------------------------------------------
// per-tile survivors of the tiled passes, then their exclusive scan
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_tile_kept(PassBufs b)
{
    // one wave per tile: a tile's window entries (a few hundred) take one
    // round of loads, and every tile's wave is resident at once
    constexpr int UN = 4;
    DevCtl *ctl = b.ctl;
    const u64 tile = (u64)blockIdx.x * 4 + (threadIdx.x >> 6); // below the tile arrays' length
    // every control load issued before any is used
    const u64 n = *b.n_in;
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const int shift = ctl->side_slab_shift, spl = ctl->side_spt_log2;
    const u64 ntiles = (n + 2047) / 2048;
    if (tile >= ntiles) return; // the whole wave
    // the tile's window entries (one slab, or one per wave of the histogram
    // pass), and its candidates certain before the cut
    const TileSlabs sd = tile_slabs(b.t_side, tile, spl, shift, false, b.side_cap);
    u64 na = 0;
    for (int w = 0; w < (1 << spl); ++w) na += b.t_above[(tile << spl) + (u64)w];
    const u32 ns = sd.n;
    const u32 lane = (u32)sts_lane();
    u32 c = 0;
    for (u32 i0 = 0; i0 < ns; i0 += UN * 64) {
        u64 w[UN], k[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            const u32 j = i0 + (u32)r * 64 + lane;
            const u64 i = j < ns ? slab_at(sd, j) : slab_at(sd, 0);
            w[r] = b.side_w[i];
            k[r] = b.side_key[i];
        }
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            const u32 j = i0 + (u32)r * 64 + lane;
            // ranked at or above the threshold term; the key decides only a tie
            c += (j < ns && (w[r] > thr_w || (w[r] == thr_w && k[r] <= thr_k))) ? 1u : 0u;
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
    if (lane == 0) b.t_off[tile] = na + c;
}

__global__ void __launch_bounds__(1024) k_tile_scan(PassBufs b)
{
    constexpr int CH = 8; // tiles per thread per round, loaded before use
    __shared__ u64 s_scratch[16];
    __shared__ u64 s_carry;
    DevCtl *ctl = b.ctl;
    const u64 n = *b.n_in;
    const u64 ntiles = (n + 2047) / 2048;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (u64 c0 = 0; c0 < ntiles; c0 += 1024ull * CH) {
        const u64 lo = c0 + (u64)threadIdx.x * CH;
        u64 v[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) v[k] = lo + k < ntiles ? b.t_off[lo + k] : 0ull;
        u64 sum = 0;
#pragma unroll
        for (int k = 0; k < CH; ++k) sum += v[k];
        u64 total;
        u64 run = block_excl_scan<u64, 1024>(sum, s_scratch, &total) + s_carry;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            if (lo + k < ntiles) b.t_off[lo + k] = run;
            run += v[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) s_carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const u64 total = s_carry;
        *b.n_out = total;
        if (total > b.out_cap) atomicOr(&ctl->flags, STS_F_OUT_OVERFLOW);
    }
}

__global__ void k_init_state(u64 *keys, double2 *amps64, float2 *amps32, u64 *n_out)
{
    keys[0] = 0;
    if (amps64) amps64[0] = make_double2(1.0, 0.0);
    if (amps32) amps32[0] = make_float2(1.0f, 0.0f);
    *n_out = 1;
}

__global__ void k_set_n(u64 *n_out, u64 n) { *n_out = n; }

// the gate's description into device memory, where every kernel of its step
// reads it (a captured step is replayed for another gate by changing this
// one launch's argument)
__global__ void __launch_bounds__(64) k_set_gate(GateArg g, GateArg *dst)
{
    static_assert(sizeof(GateArg) % sizeof(u32) == 0, "GateArg is a whole number of words");
    const u32 *src = reinterpret_cast<const u32 *>(&g);
    u32 *d = reinterpret_cast<u32 *>(dst);
    for (u32 i = threadIdx.x; i < sizeof(GateArg) / sizeof(u32); i += 64) d[i] = src[i];
}

// before the terms' buckets are counted
__global__ void __launch_bounds__(256) k_load_clear(u32 *counts, u64 n, DevCtl *ctl)
{
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) counts[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->load_most = 0;
}

// Terms from and to the host: one read of what the copy brought (bound by HBM, some
// us); sorting and checking on the host took 34 of a hand-over's 35 ms at 300,007
// terms.
// range and finiteness of n terms from the host; complex64: their amplitudes
// rounded to FP32 (nearest-even); and how many of a quarter
// of them lie in each bucket
__global__ void __launch_bounds__(256) k_load_check(const u64 *__restrict__ keys, const double2 *__restrict__ amps,
                                                    u64 n, u64 limit, float2 *amps32, int hb, u32 *counts, DevCtl *ctl)
{
    bool bad = false;
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) {
        const double2 a = amps[i];
        const u64 key = keys[i];
        bad |= key > limit || !isfinite(a.x) || !isfinite(a.y);
        if (amps32) amps32[i] = make_float2((float)a.x, (float)a.y);
        // (a quarter of the terms, by another hash: 5 us at 300,007 terms, 15 for all)
        if (counts && sts_mix64(key) >> 62 == 0) {
            u32 v = 0;
            for (int j = 0; j < hb; ++j) v |= sts_parity(key, k_lin_masks[32 - hb + j]) << j;
            atomicAdd(&counts[v], 1u);
        }
    }
    if (bad) atomicOr(&ctl->load_flags, 1u);
}

__global__ void __launch_bounds__(256) k_load_unique(const u64 *__restrict__ keys, u64 n, const u32 *__restrict__ counts,
                                                     u64 buckets, DevCtl *ctl)
{
    bool bad = false;
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x + 1; i < n; i += (u64)gridDim.x * 256)
        bad |= keys[i] == keys[i - 1];
    if (bad) atomicOr(&ctl->load_flags, 1u);
    u32 most = 0;
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < buckets; i += (u64)gridDim.x * 256)
        most = counts[i] > most ? counts[i] : most;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const u32 o = __shfl_xor(most, d, 64);
        most = o > most ? o : most;
    }
    if (sts_lane() == 0 && most) atomicMax(&ctl->load_most, most);
}

__global__ void __launch_bounds__(256) k_widen(const float2 *__restrict__ in, double2 *__restrict__ out, u64 n)
{
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256)
        out[i] = make_double2((double)in[i].x, (double)in[i].y);
}

// zero n words (a kernel rather than a memset, so the work can sit in a
// captured graph)
__global__ void __launch_bounds__(256) k_fill_zero(u64 *p, u64 n)
{
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) p[i] = 0;
}

// a fresh control block: the rule, nothing cut yet, n_in terms in buffer 0
__global__ void __launch_bounds__(64) k_ctl_begin(DevCtl *ctl, u64 K, double p, u64 n_in)
{
    u64 *w = reinterpret_cast<u64 *>(ctl);
    constexpr u64 words = sizeof(DevCtl) / sizeof(u64);
    static_assert(sizeof(DevCtl) % sizeof(u64) == 0, "DevCtl is a whole number of words");
    for (u64 i = threadIdx.x; i < words; i += 64) w[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        ctl->K = K;
        ctl->p = p;
        ctl->scale = 1.0;
        ctl->frac = 1.0;
        ctl->e_pred = -1;
        ctl->cnt[0] = n_in;
    }
}

// copy the cnt[slot] terms of (keys, amps) to the caller's arrays (at most
// out_cap), their count to *n_out and, if stats is set, W and the kept
// fraction to stats[0..1]
__global__ void __launch_bounds__(256) k_terms_out(const u64 *keys, const void *amps, int amp_bytes,
                                                   const DevCtl *ctl, int slot, u64 *keys_out, void *amps_out,
                                                   u64 out_cap, u64 *n_out, double *stats)
{
    const u64 n0 = ctl->cnt[slot];
    const u64 n = n0 < out_cap ? n0 : out_cap;
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) {
        keys_out[i] = keys[i];
        if (amp_bytes == 16) reinterpret_cast<double2 *>(amps_out)[i] = reinterpret_cast<const double2 *>(amps)[i];
        else reinterpret_cast<float2 *>(amps_out)[i] = reinterpret_cast<const float2 *>(amps)[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *n_out = n;
        if (stats) {
            stats[0] = ctl->W;
            stats[1] = ctl->frac;
        }
    }
}

} // namespace

hipError_t launch_pick1(const PassBufs &b, int groups, int peak_only, int predicted, hipStream_t s)
{
    hipLaunchKernelGGL(k_pick1, dim3(1), dim3(256), 0, s, b, groups, peak_only, predicted);
    return hipGetLastError();
}

hipError_t launch_pick_window(const PassBufs &b, int groups, hipStream_t s)
{
    hipLaunchKernelGGL(k_pick_window, dim3(1), dim3(256), 0, s, b, groups);
    return hipGetLastError();
}

hipError_t launch_side_hist(const PassBufs &b, u64 *h2, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_side_hist, dim3(grid), dim3(256), 0, s, b, h2);
    return hipGetLastError();
}

hipError_t launch_side_extract(const PassBufs &b, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_side_extract, dim3(grid), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_tile_kept(const PassBufs &b, int tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile_kept, dim3((tiles + 3) / 4), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_tile_scan(const PassBufs &b, u64 ntiles_bound, hipStream_t s)
{
    (void)ntiles_bound;
    hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_final(const PassBufs &b, hipStream_t s)
{
    hipLaunchKernelGGL(k_final, dim3(1), dim3(FT), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_init_state(int prec, u64 *keys, void *amps, u64 *n_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(1), 0, s, keys, prec == 0 ? (double2 *)amps : nullptr,
                       prec == 0 ? nullptr : (float2 *)amps, n_out);
    return hipGetLastError();
}

hipError_t launch_set_gate(const GateArg &g, GateArg *dst, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_gate, dim3(1), dim3(64), 0, s, g, dst);
    return hipGetLastError();
}

const void *set_gate_kernel() { return reinterpret_cast<const void *>(&k_set_gate); }

hipError_t launch_set_n(u64 *n_out, u64 n, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_n, dim3(1), dim3(1), 0, s, n_out, n);
    return hipGetLastError();
}

static dim3 stream_grid(u64 n) { return dim3((unsigned)std::max<u64>(1, std::min<u64>((n + 255) / 256, 2048))); }

hipError_t launch_load_check(int prec, const u64 *keys, const double *amps, u64 n, u64 limit, float2 *amps32, int hb,
                             u64 *counts, DevCtl *ctl, hipStream_t s)
{
    if (counts) hipLaunchKernelGGL(k_load_clear, stream_grid(1ull << hb), dim3(256), 0, s, (u32 *)counts, 1ull << hb,
                                   ctl);
    hipLaunchKernelGGL(k_load_check, stream_grid(n), dim3(256), 0, s, keys, (const double2 *)amps, n, limit,
                       prec == 0 ? nullptr : amps32, hb, (u32 *)counts, ctl);
    return hipGetLastError();
}

hipError_t launch_load_unique(const u64 *sorted, u64 n, int hb, const u64 *counts, DevCtl *ctl, hipStream_t s)
{
    hipLaunchKernelGGL(k_load_unique, stream_grid(n), dim3(256), 0, s, sorted, n, (const u32 *)counts,
                       counts ? 1ull << hb : 0ull, ctl);
    return hipGetLastError();
}

hipError_t launch_widen(const float2 *in, double2 *out, u64 n, hipStream_t s)
{
    hipLaunchKernelGGL(k_widen, stream_grid(n), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

hipError_t launch_fill_zero(u64 *p, u64 n, hipStream_t s)
{
    const u64 blocks = std::min<u64>((n + 255) / 256, 1024);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_ctl_begin(DevCtl *ctl, u64 K, double p, u64 n_in, hipStream_t s)
{
    hipLaunchKernelGGL(k_ctl_begin, dim3(1), dim3(64), 0, s, ctl, K, p, n_in);
    return hipGetLastError();
}

hipError_t launch_terms_out(const u64 *keys, const void *amps, int amp_bytes, const DevCtl *ctl, int slot,
                            u64 *keys_out, void *amps_out, u64 out_cap, u64 *n_out, double *stats, hipStream_t s)
{
    const u64 blocks = std::max<u64>(std::min<u64>((out_cap + 255) / 256, 1024), 1);
    hipLaunchKernelGGL(k_terms_out, dim3((unsigned)blocks), dim3(256), 0, s, keys, amps, amp_bytes, ctl, slot,
                       keys_out, amps_out, out_cap, n_out, stats);
    return hipGetLastError();
}
