// tiny_impl.h - the gate step of a state of at most STS_TINY_MAX terms (gates
// of 1 and 2 qubits) in one launch of one workgroup.
//
// Such a step is all latency: in a chain of launches it spends some 10 us each
// on a dozen of them, whatever its size. Here the terms are grouped in one
// hash table in LDS, every thread keeps its groups' candidates (key, amplitude,
// weight) in registers from the product to the write, and all of the
// selection (exponent bins, level picks, the exact cut) runs on LDS. The state
// needs no particular order; the survivors are written in the order of their
// groups' first members. 11 us at 1,024 complex128 terms, where the chain took 116.
#pragma once
#include "group_impl.h"
#include "select_impl.h"

namespace sts_tiny {

using namespace sts_group;
using namespace sts_select;

// Two terms per thread, in the smallest workgroup that holds the state: what
// the one CU spends is its waves times the instructions of each.
constexpr int RPT = 2;

// exponent bins in LDS: sums of mantissa >> 26; & (2^26 - 1), plus count << 44
struct LdsBins {
    u64 *s_hi, *s_lo;
    __device__ __forceinline__ void load(int, int e, u64 &c, u64 &hi, u64 &lo) const
    {
        c = s_lo[e] >> 44;
        hi = s_hi[e];
        lo = s_lo[e] & ((1ull << 44) - 1);
    }
    __device__ __forceinline__ void clear(int) const {}
};

template <typename AT, int NT> struct TinySmem {
    static constexpr int CAP = RPT * NT, SLOTS = 2 * CAP;
    union {
        struct {
            AT amp[CAP];
            u64 key[CAP];
            unsigned long long slot[SLOTS]; // a group: the index + 1 of its member j at bit 16 j
        } g;
        Level1Smem<NT> l1;
        __attribute__((aligned(16))) unsigned char raw[THIN_BINS * 12];
    } u;
    u64 hi[STS_NBIN], lo[STS_NBIN];
    Level1Cut l1;
    CutSmem cut;
    Sub sub;
    u32 scan[NT / 64];
};

template <typename AT, int M, int NT>
__global__ void __launch_bounds__(NT) k_tiny(GateArg g, PassBufs b)
{
    typedef typename Scalar<AT>::T R;
    constexpr int NP = 1 << M;
    constexpr int CAP = TinySmem<AT, NT>::CAP, SLOTS = TinySmem<AT, NT>::SLOTS;
    __shared__ TinySmem<AT, NT> s;
    DevCtl *ctl = b.ctl;
    const int t = threadIdx.x;
    const u64 nm = g.notmask;
    const u64 K = ctl->K;
    const double l10 = ctl->log10_cum;
    const u32 n = (u32)*b.n_in; // at most CAP (the host's bound)
    const AT *amps = (const AT *)b.amps;
    u64 key[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const u32 i = (u32)(r * NT + t);
        if (i < n && i < CAP) {
            key[r] = b.keys[i];
            s.u.g.key[i] = key[r];
            s.u.g.amp[i] = amps[i];
        }
    }
    for (int i = t; i < SLOTS; i += NT) s.u.g.slot[i] = 0;
    for (int i = t; i < STS_NBIN; i += NT) {
        s.hi[i] = 0;
        s.lo[i] = 0;
    }
    __syncthreads();
    // open addressing on the masked key; every member's pattern is its own,
    // so the members of a group never collide in its word
    u32 at[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const u32 i = (u32)(r * NT + t);
        if (i < n && i < CAP) {
            const u64 rest = key[r] & nm;
            u32 j = 0;
#pragma unroll
            for (int q = 0; q < M; ++q) j |= (u32)((key[r] >> g.q[q]) & 1ull) << q;
            const unsigned long long mine = (unsigned long long)(i + 1) << (16 * j);
            u32 h = (u32)(((u32)rest * 0x9e3779b1u + (u32)(rest >> 32) * 0x85ebca6bu) >> 20) & (SLOTS - 1);
            for (;;) {
                const unsigned long long old = atomicCAS(&s.u.g.slot[h], 0ull, mine);
                if (old == 0) break;
                const int f = (__ffsll((long long)old) - 1) & ~15;
                if ((s.u.g.key[(u32)((old >> f) & 0xffffu) - 1u] & nm) == rest) {
                    atomicOr(&s.u.g.slot[h], mine);
                    break;
                }
                h = (h + 1) & (SLOTS - 1);
            }
            at[r] = h;
        }
    }
    __syncthreads();
    // the first member (in the state's order) leads its group
    u64 rest[RPT];
    R ox[RPT][NP], oy[RPT][NP];
    auto weight = [&](int r, int p) { // recomputed at each use: registers are what this kernel is short of
        AT o;
        o.x = ox[r][p];
        o.y = oy[r][p];
        return weight_bits(o);
    };
    u32 cand = 0; // a bit per round and pattern
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const u32 i = (u32)(r * NT + t);
        Group<AT, M> G;
        G.present = 0;
        group_clear<AT, M>(G);
        rest[r] = 0;
        if (i < n && i < CAP) {
            const unsigned long long word = s.u.g.slot[at[r]];
            bool lead = true;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const u32 k = (u32)((word >> (16 * j)) & 0xffffu);
                lead = lead && (k == 0 || k >= i + 1);
            }
            if (lead) {
                rest[r] = key[r] & nm;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const u32 k = (u32)((word >> (16 * j)) & 0xffffu);
                    if (k) {
                        G.v[j] = s.u.g.amp[k - 1];
                        G.present |= 1u << j;
                    }
                }
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const AT o = group_out<AT, M>(g, G, p);
            ox[r][p] = o.x;
            oy[r][p] = o.y;
            if (G.present && nonzero(o)) {
                cand |= 1u << (r * NP + p);
                if (!b.materialise) {
                    const u64 w = weight_bits(o);
                    const u64 mant = sts_mant(w);
                    const u32 e = (u32)(w >> 52);
                    // (at most 2^13 candidates: neither field overflows)
                    atomicAdd((unsigned long long *)&s.hi[e], mant >> 26);
                    atomicAdd((unsigned long long *)&s.lo[e], (mant & ((1ull << 26) - 1)) | (1ull << 44));
                }
            }
        }
    }
    __syncthreads();
    bool all = b.materialise;
    u64 thr_w = 0, thr_k = 0;
    if (!all) {
        pick_level1<NT>(b, 0, 0, 0, s.u.l1, LdsBins{s.hi, s.lo});
        __syncthreads();
        if (t < (int)(sizeof(Level1Cut) / sizeof(u64)))
            reinterpret_cast<u64 *>(&s.l1)[t] = reinterpret_cast<const u64 *>(&s.u.l1.cut)[t];
        __syncthreads();
        all = s.l1.keep_all;
    }
    const bool cut = !all;
    if (cut) {
        const int e = s.l1.e;
        if (t == 0) {
            s.sub.cnt_before = s.l1.cnt;
            s.sub.mb = 0;
            s.sub.vpre = 0;
            s.sub.vshift = 116;
            s.sub.count = s.l1.count;
        }
        __syncthreads();
        auto each = [&](int vshift, u128 vpre, bool, auto f) {
#pragma unroll
            for (int r = 0; r < RPT; ++r)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const u64 w = weight(r, p);
                    if (!((cand >> (r * NP + p)) & 1u) || (int)(w >> 52) != e) continue;
                    const u128 v = rank_key(w, rest[r] | g.dep[p]);
                    if ((v >> vshift) == vpre) f(v);
                }
        };
        if (!resolve_cut<NT, true>(each, e, K, make128(s.l1.R_lo, s.l1.R_hi), s.sub, s.u.raw, s.cut)) { // uniform
            if (t == 0) { // (an internal inconsistency: reported, and no term kept)
                atomicOr(&ctl->flags, STS_F_UNRESOLVED);
                *b.n_out = 0;
            }
            return;
        }
        thr_w = s.cut.thr_w;
        thr_k = s.cut.thr_k;
        if (t >= NT - 64) finish_cut(ctl, s.cut, e, s.l1.S, s.l1.total, s.l1.W, l10);
    }
    u32 keep = 0;
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const u64 k = rest[r] | g.dep[p], w = weight(r, p);
            const bool in = ((cand >> (r * NP + p)) & 1u) && (!cut || w > thr_w || (w == thr_w && k <= thr_k));
            keep |= in ? 1u << (r * NP + p) : 0u;
        }
    u32 base = 0, pos[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        u32 tot; // (the scans' barriers also publish the scale)
        pos[r] = base + block_excl_scan<u32, NT>((u32)__popc((keep >> (r * NP)) & ((1u << NP) - 1u)), s.scan, &tot);
        base += tot;
    }
    const bool rescale = cut && s.cut.dropped;
    const double scale = rescale ? s.cut.scale : 1.0;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (!((keep >> (r * NP + p)) & 1u)) continue;
            if (pos[r] < b.out_cap) {
                AT o;
                o.x = ox[r][p];
                o.y = oy[r][p];
                b.out_keys[pos[r]] = rest[r] | g.dep[p];
                ((AT *)b.out_amps)[pos[r]] = out_amp(o, rescale, scale);
            }
            ++pos[r];
        }
    }
    if (t == 0) {
        *b.n_out = base;
        if (base > b.out_cap) atomicOr(&ctl->flags, STS_F_OUT_OVERFLOW);
    }
}

template <typename AT, int M> const void *kernel(int size)
{
    return size == 0 ? reinterpret_cast<const void *>(&k_tiny<AT, M, 256>)
                     : size == 1 ? reinterpret_cast<const void *>(&k_tiny<AT, M, 512>)
                                 : reinterpret_cast<const void *>(&k_tiny<AT, M, 1024>);
}

template <typename AT, int M> hipError_t launch(const GateArg &g, const PassBufs &b, u64 n_bound, hipStream_t s)
{
    static_assert(STS_TINY_MAX == RPT * 1024, "the largest workgroup's terms");
    if (n_bound <= RPT * 256) hipLaunchKernelGGL((k_tiny<AT, M, 256>), dim3(1), dim3(256), 0, s, g, b);
    else if (n_bound <= RPT * 512) hipLaunchKernelGGL((k_tiny<AT, M, 512>), dim3(1), dim3(512), 0, s, g, b);
    else hipLaunchKernelGGL((k_tiny<AT, M, 1024>), dim3(1), dim3(1024), 0, s, g, b);
    return hipGetLastError();
}

} // namespace sts_tiny
