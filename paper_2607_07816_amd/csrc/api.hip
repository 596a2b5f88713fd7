// api.hip - the C ABI of libsts: context, device memory, and the order in
// which the kernels of a gate step run.
//
// A gate step (sts_apply_gate then sts_truncate) runs on the context's stream
// and without host synchronisation. Which kernels depends on the size bound:
//   up to 2048 terms (gates of 1 and 2 qubits): one launch (tiny_impl.h);
//   more, gates of 1 and 2 qubits: the state is kept in the order of a linear
//   hash of its keys (linhash.h), in which a gate's partners and new terms
//   share four buckets, so that nothing is sorted (bucket_impl.h):
//     up to 2^17 terms: weigh all candidates (above 2^14 after a pass that
//     finds the window), select in one workgroup, write;
//     above: sample a window, weigh, decide and pick, list and resolve the
//     last terms, count and place the survivors, write; further passes that
//     exit at once unless the window missed;
//   gates of 3 qubits and more, and the one step of sts_step_static:
//   1. 1..4 radix digit passes (per-tile counts, per-digit scan, scatter):
//      group the state by the hash bucket of the bits outside the gate
//      (radix.hip);
//   2. histogram pass: recompute every new amplitude, histogram its weight by
//      exponent field with exact mantissa sums (group.hip);
//   3. level-1 pick: exact prefix over exponent bins (select.hip);
//   4. extraction pass: copy the candidates of the cut's exponent to the side
//      buffer (group.hip);
//   5. level-2 histogram + pick over the side buffer, then the final levels
//      and the ranking of the last <= 128 candidates (select.hip);
//   6. write pass: recompute once more and write the survivors, rescaled
//      (group.hip).
// Without a truncation rule (or when the next gate arrives first) the write
// alone runs, keeping every nonzero candidate.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "sts.h"
#include "kernels.h"

namespace {

constexpr u64 kAlign = 256;
constexpr int kULen = 32 * 32 * 2; // doubles of the largest U

u64 align_up(u64 x) { return (x + kAlign - 1) & ~(kAlign - 1); }

u64 ceil_div(u64 a, u64 b) { return (a + b - 1) / b; }

struct Layout {
    u64 ctl, ctl_save, keys[3], amps[3], side_key, side_w, side_amp, sub_key, sub_w, h1, h2, h2w, h3, best, rcount, rprefix, rtotal, look_comp,
        t_above, t_side, t_off, w_all, w_kept, t_base, bd[2], tctr, dU, sub_cnt, wpart, sbins, gate, total;
};

// tiles of the LDS-tiled passes (2048 terms each) and the side-buffer entries:
// one slab of 2048 << m entries per tile, m <= 3
u64 tiled_tiles(u64 cap) { return (cap + 2047) / 2048 + 1; }
u64 side_capacity(u64 cap) { return tiled_tiles(cap) * (2048ull << 3); }

// Bucket bits of a state of at most n terms. A wave's share is four buckets:
// 128 to 256 terms of a large state, so that its runs are at least 256 bytes
// long and its rounds of 64 lanes are full; of a state of less than 2^20 terms
// rather 32 to 64, so that there are shares for every CU's waves.
int bucket_bits(u64 n)
{
    int lg = 0;
    while ((1ull << lg) < n && lg < 63) ++lg;
    return std::max(lg <= 18 ? lg - 4 : std::max(14, lg - 6), STS_BKT_DIMS);
}

// largest state that is kept in bucket order (32-bit term indices, and bucket
// tables of at most 2^22 entries)
constexpr u64 kBucketMax = 1ull << 28;
// Up to this size bound a step's selection is one workgroup's (k_bkt_select);
// above, the step samples its window and spreads the selection over many
// launches. At 131,072 terms a step took 87 us instead of 93 (complex128: 89
// and 89), at 65,536 67 instead of 89; that workgroup's lists hold no more shares.
constexpr u64 kSelectMax = 1ull << 17;
// Up to this one that workgroup reads a window of two octaves around the
// previous cut; above, one bin that a pass over all terms has found. At 16,384
// terms 51 us instead of 54, at 32,768 69 and 59.
constexpr u64 kSmallMax = 1ull << 14;

// Terms from the host of which a quarter has this many in one bucket (of 2 to
// 16 on average, and up to 36 by chance) take the sort: a share of four buckets
// of 160 terms and more no longer fits a wave's tables twice, and larger ones are
// scanned once for each of their parts. Steps of 60,000 terms with 117 in a bucket:
// 62 us bucketed, 154 sorted; with 234: 1610 and 176. Of 150,000 with 146: 136 and
// 192, with 293 262 and 190. Of 2^20 with 128: 396 and 236, with 1024 8650 and 245.
constexpr u32 kCrowded = 48;

Layout make_layout(u64 cap, int prec)
{
    const u64 asz = prec == STS_C128 ? 16 : 8;
    const u64 scap = side_capacity(cap);
    const u64 ttiles = tiled_tiles(cap);
    const u64 tiles = ceil_div(cap, 2048) + 1; // the smallest grouping-sort tile
    const u64 gtiles = ceil_div(cap, STS_GTILE);
    Layout L;
    u64 o = 0;
    auto take = [&](u64 bytes) {
        const u64 at = o;
        o = align_up(o + bytes);
        return at;
    };
    L.ctl = take(sizeof(DevCtl));
    L.ctl_save = take(sizeof(DevCtl));
    for (int i = 0; i < 3; ++i) L.keys[i] = take(cap * 8);
    for (int i = 0; i < 3; ++i) L.amps[i] = take(cap * asz);
    L.side_key = take(scap * 8);
    L.side_w = take(scap * 8);
    L.side_amp = take(scap * asz);
    L.sub_key = take((u64)STS_SUB_CAP * 8);
    L.sub_w = take((u64)STS_SUB_CAP * 8);
    L.h1 = take(3 * STS_NBIN * 8);
    L.h2 = take(3 * STS_NBIN * 8);
    L.h2w = take(3 * STS_NBIN * 8);
    L.h3 = take(3 * STS_NBIN * 8);
    L.best = take(2 * STS_MAX_GROUPS * 8);
    L.rcount = take(2048 * tiles * 4); // per digit (up to 11-bit digits) and tile
    L.rprefix = take(2048 * tiles * 8);
    L.rtotal = take(2048 * 8);
    L.look_comp = take(gtiles * 8);
    const u64 buckets = cap <= kBucketMax ? 1ull << bucket_bits(cap) : 0;
    const u64 slabs = std::max(ttiles * 4, buckets / 4); // up to 4 slabs per tile
    L.t_above = take(slabs * 4);
    L.t_side = take(slabs * 4);
    L.t_off = take(std::max(ttiles, buckets / 16) * 8);
    L.w_all = take(buckets);  // a word per share of four buckets
    L.w_kept = take(buckets);
    L.t_base = take((buckets / 16 / STS_BKT_CHUNK + 1) * 8);
    for (int i = 0; i < 2; ++i) L.bd[i] = take(buckets * sizeof(uint2));
    L.tctr = take(16 * 4);
    L.dU = take(kULen * 8 + kULen * 4); // U in FP64, then its FP32 rounding
    L.sub_cnt = take((STS_SUB_REGIONS + 1) * 128);
    L.wpart = take(9 * STS_MAX_GROUPS * 8);
    L.sbins = take(STS_SW_WORDS * 8);
    L.gate = take(2 * sizeof(GateArg)); // the current gate, and the identity
    L.total = o;
    return L;
}

// the working memory of sts_step_static: one array per device, holding a
// context laid out for STS_STATIC_MAX_TERMS terms of either precision
constexpr size_t kStaticBytes = 32ull << 20;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

// its address on the current device (the array's name is a host-side
// stand-in, never a device address); looked up once per device
hipError_t static_scratch(void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

} // namespace

struct sts_ctx {
    int n_qubits = 0;
    int prec = 0;
    u64 K = 0;
    double p = 0.0;
    hipStream_t stream = nullptr;
    bool own_mem = false;
    unsigned char *mem = nullptr;
    u64 cap = 0, scap = 0, tiles_cap = 0, gtiles_cap = 0;
    u64 *keys[3] = {nullptr, nullptr, nullptr};
    void *amps[3] = {nullptr, nullptr, nullptr};
    int cur = 0;            // buffer with the state, or the sorted input of the pending gate
    int radix_small_log2 = 0;               // states of at most 2^this terms are sorted with
    int radix_small_shape = STS_RADIX_8x16; // this shape; larger ones with 8x16
    bool pending = false;   // a gate whose new amplitudes are not written yet
    GateArg gate;
    u64 n_bound = 1;        // upper bound on the terms in buffer cur
    DevCtl *ctl = nullptr;
    DevCtl *ctl_save = nullptr; // the control block as it was before a step that may be refused
    u64 *h1 = nullptr, *h2 = nullptr, *h2w = nullptr, *h3 = nullptr, *best = nullptr;
    u64 *side_key = nullptr, *side_w = nullptr, *sub_key = nullptr, *sub_w = nullptr;
    void *side_amp = nullptr;
    u32 *rcount = nullptr;                          // per-tile digit counts of a scatter pass
    u64 *rprefix = nullptr, *rtotal = nullptr, *look_comp = nullptr;
    u32 *t_above = nullptr, *t_side = nullptr;
    u64 *t_off = nullptr;
    u32 *w_all = nullptr, *w_kept = nullptr;
    u64 *t_base = nullptr;
    uint2 *bd[2] = {nullptr, nullptr}; // bucket tables
    bool crowded = false;   // loaded terms that crowd in few buckets: not kept in bucket order
    bool bucketed = false;  // the state in buffer cur is in bucket order:
    int hb = 0, bdc = 0;    // 2^hb buckets, table bd[bdc]
    bool one_step = false;    // sts_step_static
    bool bkt_pending = false; // the pending gate is a bucketed step
    bool tiny_pending = false; // or a one-launch step
    int prev_m = 0, prev_q[2] = {0, 0}; // the qubits of the last bucketed step
    u32 *tctr = nullptr;
    double *dU = nullptr;
    u32 *sub_cnt = nullptr;
    u64 *wpart = nullptr, *sbins = nullptr;
    GateArg *dgate = nullptr, *dgate_id = nullptr; // device copies of the gate and of the identity
    const GateArg *gate_dev = nullptr;              // the one the pending step's kernels read
    double *hU = nullptr;    // pinned staging of U for m >= 4
    hipEvent_t u_event = nullptr;
    bool u_event_live = false;
    DevCtl *hctl = nullptr;  // pinned mirror of the control block
    u32 epoch = 0;
    bool poisoned = false;
    // optional per-kernel timing
    bool prof = false;
    struct Mark {
        int kind;
        hipEvent_t a, b;
    };
    std::vector<Mark> marks;
    std::vector<hipEvent_t> pool;
    double prof_ms[STS_K_COUNT] = {};
    u64 prof_n[STS_K_COUNT] = {};
};

namespace {

sts_status fail_hip(sts_ctx *c, hipError_t e)
{
    if (e == hipSuccess) return STS_OK;
    if (c) c->poisoned = true;
    return e == hipErrorOutOfMemory ? STS_E_NOMEM : STS_E_HIP;
}

#define STS_TRY(c, expr)                                   \
    do {                                                   \
        const hipError_t _e = (expr);                      \
        if (_e != hipSuccess) return fail_hip((c), _e);    \
    } while (0)

hipEvent_t prof_event(sts_ctx *c)
{
    if (!c->pool.empty()) {
        hipEvent_t e = c->pool.back();
        c->pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// a kernel launch, bracketed by events when timing is on
#define STS_LAUNCH(c, kind, expr)                                                  \
    do {                                                                           \
        hipEvent_t _a = nullptr, _b = nullptr;                                     \
        if ((c)->prof) {                                                           \
            _a = prof_event(c);                                                    \
            _b = prof_event(c);                                                    \
            if (_a && _b) STS_TRY(c, hipEventRecord(_a, (c)->stream));             \
        }                                                                          \
        STS_TRY(c, expr);                                                          \
        if (_a && _b) {                                                            \
            STS_TRY(c, hipEventRecord(_b, (c)->stream));                           \
            (c)->marks.push_back({(kind), _a, _b});                                \
        }                                                                          \
    } while (0)

// fold finished marks into the per-kind totals (after a synchronisation)
void prof_collect(sts_ctx *c)
{
    for (auto &m : c->marks) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, m.a, m.b) == hipSuccess) {
            c->prof_ms[m.kind] += ms;
            c->prof_n[m.kind] += 1;
        }
        c->pool.push_back(m.a);
        c->pool.push_back(m.b);
    }
    c->marks.clear();
}

u32 next_epoch(sts_ctx *c)
{
    if (++c->epoch >= (1u << 24)) {
        // tags wrap: clear every look-back word once
        (void)hipMemsetAsync(c->look_comp, 0, c->gtiles_cap * 8, c->stream);
        c->epoch = 1;
    }
    return c->epoch;
}

u64 sat_shl(u64 x, int m)
{
    if (m <= 0) return x;
    if (x > (~0ull >> m)) return ~0ull;
    return x << m;
}

PassBufs pass_bufs(sts_ctx *c, int in, int out)
{
    PassBufs b;
    std::memset(&b, 0, sizeof(b));
    b.gate = c->gate_dev;
    b.gate_dst = c->dgate;
    b.keys = c->keys[in];
    b.amps = c->amps[in];
    b.n_in = &c->ctl->cnt[in];
    b.n_out = out >= 0 ? &c->ctl->cnt[out] : nullptr;
    b.ctl = c->ctl;
    b.h1 = c->h1;
    b.h2w = c->h2w;
    b.h3 = c->h3;
    b.best = c->best;
    b.side_key = c->side_key;
    b.side_w = c->side_w;
    b.side_amp = c->side_amp;
    b.side_cap = c->scap;
    b.sub_key = c->sub_key;
    b.sub_w = c->sub_w;
    b.sub_cap = STS_SUB_CAP;
    b.sub_cnt = c->sub_cnt;
    if (out >= 0) {
        b.out_keys = c->keys[out];
        b.out_amps = c->amps[out];
    }
    b.out_cap = c->cap;
    b.look = c->look_comp;
    b.t_above = c->t_above;
    b.t_side = c->t_side;
    b.t_off = c->t_off;
    b.w_all = c->w_all;
    b.w_kept = c->w_kept;
    b.t_base = c->t_base;
    b.bd_in = c->bd[c->bdc];
    b.bd_out = c->bd[c->bdc ^ 1];
    b.tile_ctr = c->tctr + 4;
    b.wpart = c->wpart;
    b.sbins = c->sbins;
    return b;
}

// whether a gate of m qubits takes the LDS-tiled passes: always for m <= 3;
// for m = 4 when every tile's side slab (2048 << 4 entries) fits the side
// buffer, i.e. when the state holds at most about half the capacity
bool use_tiles(const sts_ctx *c, int m)
{
    if (m <= 3) return true;
    if (m > 4) return false;
    return ceil_div(std::max<u64>(c->n_bound, 1), 2048) * (2048ull << 4) <= c->scap;
}

// workgroups of the histogram pass (persistent; the tiled pass walks
// 2048-term tiles), at most as many as are resident at once
int hist_groups(int prec, u64 n_bound, int m, bool tiled)
{
    const u64 g = ceil_div(n_bound ? n_bound : 1, tiled ? 2048 : STS_WG);
    const u64 cap = (u64)std::min(group_hist_capacity(prec, m, tiled), STS_MAX_GROUPS);
    return (int)std::min<u64>(std::max<u64>(g, 1), cap);
}

int compact_tiles(u64 n_bound, int m) { return (int)sts_compact_groups(n_bound, m); }

// point every buffer of the context into its device memory c->mem
void bind_layout(sts_ctx *c, const Layout &L)
{
    c->ctl = (DevCtl *)(c->mem + L.ctl);
    c->ctl_save = (DevCtl *)(c->mem + L.ctl_save);
    for (int i = 0; i < 3; ++i) {
        c->keys[i] = (u64 *)(c->mem + L.keys[i]);
        c->amps[i] = c->mem + L.amps[i];
    }
    c->side_key = (u64 *)(c->mem + L.side_key);
    c->side_w = (u64 *)(c->mem + L.side_w);
    c->side_amp = (void *)(c->mem + L.side_amp);
    c->sub_key = (u64 *)(c->mem + L.sub_key);
    c->sub_w = (u64 *)(c->mem + L.sub_w);
    c->h1 = (u64 *)(c->mem + L.h1);
    c->h2 = (u64 *)(c->mem + L.h2);
    c->h2w = (u64 *)(c->mem + L.h2w);
    c->h3 = (u64 *)(c->mem + L.h3);
    c->best = (u64 *)(c->mem + L.best);
    c->rcount = (u32 *)(c->mem + L.rcount);
    c->rprefix = (u64 *)(c->mem + L.rprefix);
    c->rtotal = (u64 *)(c->mem + L.rtotal);
    c->look_comp = (u64 *)(c->mem + L.look_comp);
    c->t_above = (u32 *)(c->mem + L.t_above);
    c->t_side = (u32 *)(c->mem + L.t_side);
    c->t_off = (u64 *)(c->mem + L.t_off);
    c->w_all = (u32 *)(c->mem + L.w_all);
    c->w_kept = (u32 *)(c->mem + L.w_kept);
    c->t_base = (u64 *)(c->mem + L.t_base);
    for (int i = 0; i < 2; ++i) c->bd[i] = (uint2 *)(c->mem + L.bd[i]);
    c->tctr = (u32 *)(c->mem + L.tctr);
    c->dU = (double *)(c->mem + L.dU);
    c->sub_cnt = (u32 *)(c->mem + L.sub_cnt);
    c->wpart = (u64 *)(c->mem + L.wpart);
    c->sbins = (u64 *)(c->mem + L.sbins);
    c->dgate = (GateArg *)(c->mem + L.gate);
    c->dgate_id = c->dgate + 1;
    c->gate_dev = c->dgate_id;
}

// copy the control block to the host and wait; map device-side error flags
sts_status sync_ctl(sts_ctx *c)
{
    STS_TRY(c, hipMemcpyAsync(c->hctl, c->ctl, sizeof(DevCtl), hipMemcpyDeviceToHost, c->stream));
    STS_TRY(c, hipStreamSynchronize(c->stream));
    // the host's checks keep every write inside its buffer and every cut
    // resolvable, so a flag here is an internal inconsistency
    if (c->hctl->flags & (STS_F_SIDE_OVERFLOW | STS_F_OUT_OVERFLOW | STS_F_UNRESOLVED)) {
        c->poisoned = true;
        return STS_E_STATE;
    }
    return STS_OK;
}

// a gate step that may still be refused for capacity keeps a copy of the
// control block (term counts, statistics, the previous cut) on the device
sts_status save_ctl(sts_ctx *c)
{
    STS_TRY(c, hipMemcpyAsync(c->ctl_save, c->ctl, sizeof(DevCtl), hipMemcpyDeviceToDevice, c->stream));
    return STS_OK;
}

// refuse the pending gate step: the control block goes back to the saved
// copy, and the state is the sorted input, i.e. the terms before the gate
sts_status refuse_step(sts_ctx *c)
{
    STS_TRY(c, hipMemcpyAsync(c->ctl, c->ctl_save, sizeof(DevCtl), hipMemcpyDeviceToDevice, c->stream));
    STS_TRY(c, hipStreamSynchronize(c->stream));
    c->pending = c->bkt_pending = false;
    return STS_E_CAPACITY;
}

// the grouping sort's shape for the state's size bound (the context's
// policy), and its digit passes: enough bucket bits for that bound
int sort_shape(const sts_ctx *c)
{
    return c->radix_small_log2 > 0 && c->n_bound <= (1ull << c->radix_small_log2) ? c->radix_small_shape
                                                                                  : STS_RADIX_8x16;
}

int sort_passes(const sts_ctx *c)
{
    const u64 nb = std::max<u64>(c->n_bound, 2);
    int lg = 0;
    while ((1ull << lg) < nb && lg < 63) ++lg;
    const int bits = sts_radix_bits(sort_shape(c));
    return std::min(std::max((lg + bits - 1) / bits, 1), 32 / bits);
}

// group the state in buffer cur by the hash bucket of key & notmask (the
// device gate's); returns
// the buffer that holds the sorted terms and the bucket bits used
sts_status sort_state(sts_ctx *c, const u64 *notmask, int *sorted, int *hb_out)
{
    const u64 nb = std::max<u64>(c->n_bound, 2);
    const int shape = sort_shape(c);
    const int bits = sts_radix_bits(shape);
    const int npass = sort_passes(c);
    const int hb = bits * npass;
    const int tiles = (int)std::max<u64>(ceil_div(nb, sts_radix_tile(shape)), 1);
    const int a = (c->cur + 1) % 3, b = (c->cur + 2) % 3;
    int src = c->cur, dst = a;
    for (int p = 0; p < npass; ++p) {
        const int shift = 64 - hb + bits * p;
        for (int what = 0; what < 3; ++what) {
            const int kind = what == 0 ? STS_K_RADIX_HIST : (what == 1 ? STS_K_RADIX_SCAN : STS_K_RADIX_PASS);
            STS_LAUNCH(c, kind, launch_radix(what, STS_SORT_BY_MIX, shape, c->prec, c->keys[src], c->amps[src],
                                             c->keys[dst], c->amps[dst], &c->ctl->cnt[src], &c->ctl->cnt[dst], notmask, shift,
                                             c->rcount, c->rprefix, c->rtotal, c->tiles_cap, tiles, c->stream));
        }
        src = dst;
        dst = dst == a ? b : a;
    }
    *sorted = src;
    *hb_out = hb;
    return STS_OK;
}

// sort n terms by key, from *k and *a through the buffers kb and ab in turn (the
// input stays as it is unless no pass is needed); *k and *a: where they end up.
// 8-bit digits at every size: a load and a read of 100,000 terms of 24 qubits
// took 440 us, 478 with 11-bit digits and one pass fewer (of 48 qubits 561 and 576)
sts_status sort_by_key(sts_ctx *c, u64 n, int prec, u64 **k, void **a, std::array<u64 *, 2> kb,
                       std::array<void *, 2> ab, const u64 *count)
{
    const int shape = STS_RADIX_8x16;
    const int bits = sts_radix_bits(shape);
    const int tiles = (int)ceil_div(n, sts_radix_tile(shape));
    for (int p = 0; p * bits < c->n_qubits; ++p) {
        for (int what = 0; what < 3; ++what)
            STS_TRY(c, launch_radix(what, STS_SORT_BY_KEY, shape, prec, *k, *a, kb[p & 1], ab[p & 1], count,
                                    &c->ctl->cnt[3], nullptr, p * bits, c->rcount, c->rprefix, c->rtotal,
                                    c->tiles_cap, tiles, c->stream));
        *k = kb[p & 1];
        *a = ab[p & 1];
    }
    return STS_OK;
}

// Terms that the host itself puts in order and checks: as many as take it less
// time than the launches of the device's passes, of which there is one per 8 key
// bits. Read and load of 256 terms of 40 qubits 64 and 36 us (on the device 146 and
// 130), of 3,000 150 and 128 (170 and 144), of 4,096 194 and 163 (174 and 151); of
// 64 qubits 4,096 192 and 163 (229 and 204), of 24 qubits 2,048 127 and 93 (136 and
// 114), 3,000 150 and 128 (135 and 112).
constexpr u64 kHostTerms = 1024 + 512 * 8;
bool on_host(const sts_ctx *c, u64 n) { return n <= 1024 + 512 * ceil_div((u64)c->n_qubits, 8); }

// n terms of the current state to the caller, in key order
sts_status read_small(sts_ctx *c, u64 n, uint64_t *keys, double *amps)
{
    u64 k[kHostTerms];
    double a[2 * kHostTerms];
    unsigned short order[kHostTerms];
    STS_TRY(c, hipMemcpyAsync(k, c->keys[c->cur], n * 8, hipMemcpyDeviceToHost, c->stream));
    STS_TRY(c, hipMemcpyAsync(a, c->amps[c->cur], n * (c->prec == STS_C128 ? 16 : 8), hipMemcpyDeviceToHost, c->stream));
    STS_TRY(c, hipStreamSynchronize(c->stream));
    for (u64 i = 0; i < n; ++i) order[i] = (unsigned short)i;
    std::sort(order, order + n, [&](unsigned short x, unsigned short y) { return k[x] < k[y]; });
    for (u64 i = 0; i < n; ++i) {
        const u64 at = order[i];
        keys[i] = k[at];
        for (u64 x = 0; x < 2; ++x) {
            float f;
            std::memcpy(&f, reinterpret_cast<const char *>(a) + (2 * at + x) * sizeof(float), sizeof(float));
            amps[2 * i + x] = c->prec == STS_C128 ? a[2 * at + x] : (double)f;
        }
    }
    return STS_OK;
}

// the bucket hash by bytes of the key
struct LinTable {
    u32 t[8][256];
    LinTable()
    {
        for (int b = 0; b < 8; ++b)
            for (int v = 0; v < 256; ++v) {
                t[b][v] = 0;
                for (int q = 0; q < 8; ++q) t[b][v] ^= (v >> q) & 1 ? lin_dir(8 * b + q) : 0u;
            }
    }
    u32 operator()(u64 key) const
    {
        u32 h = 0;
        for (int b = 0; b < 8; ++b) h ^= t[b][(key >> (8 * b)) & 255];
        return h;
    }
};

// n terms from the caller to the free buffer dst, checked before anything is
// copied; *most: the most of a quarter of them in one bucket
sts_status load_small(sts_ctx *c, u64 n, const uint64_t *keys, const double *amps, u64 limit, int dst, u32 *most)
{
    static const LinTable hash;
    u64 sorted[kHostTerms];
    for (u64 i = 0; i < n; ++i) {
        if (keys[i] > limit || !std::isfinite(amps[2 * i]) || !std::isfinite(amps[2 * i + 1])) return STS_E_ARG;
        sorted[i] = keys[i];
    }
    std::sort(sorted, sorted + n);
    for (u64 i = 1; i < n; ++i)
        if (sorted[i] == sorted[i - 1]) return STS_E_ARG;
    const int hb = bucket_bits(n);
    unsigned short counts[1 << 9] = {};
    static_assert(kHostTerms <= 1 << 13, "at most 2^9 buckets");
    *most = 0;
    for (u64 i = 0; i < n / 4; ++i) { // (any of them that are spread out)
        const u64 at = (((i * 0x9e3779b97f4a7c15ull) >> 32) * n) >> 32;
        *most = std::max<u32>(*most, ++counts[hash(keys[at]) >> (32 - hb)]);
    }
    float af[2 * kHostTerms];
    const void *src = amps;
    if (c->prec == STS_C64) {
        for (u64 i = 0; i < 2 * n; ++i) af[i] = (float)amps[i];
        src = af;
    }
    STS_TRY(c, hipMemcpyAsync(c->keys[dst], keys, n * 8, hipMemcpyHostToDevice, c->stream));
    STS_TRY(c, hipMemcpyAsync(c->amps[dst], src, n * (c->prec == STS_C128 ? 16 : 8), hipMemcpyHostToDevice, c->stream));
    STS_TRY(c, hipStreamSynchronize(c->stream)); // the caller's arrays have been read
    return STS_OK;
}

// whether a gate of m qubits on the current state is a one-launch step: at
// 2,048 terms, the most that one workgroup's LDS and registers hold, 33 us
// (with the gap to the next step) instead of 43 as a bucketed step, at 1,024 21
bool use_tiny(const sts_ctx *c, int m) { return m <= 2 && c->n_bound <= STS_TINY_MAX; }

// whether it is a bucketed step (not the one step of sts_step_static: putting its terms in bucket order
// costs what the sort does, and no later step gains from it)
bool use_buckets(const sts_ctx *c, int m)
{
    return !c->one_step && !c->crowded && m <= 2 && c->cap <= kBucketMax && c->n_bound > STS_TINY_MAX;
}

// whether the state's buckets suit its size bound: neither so few that a
// share overflows a wave's tables nor so many that they hold a handful
bool buckets_suit(const sts_ctx *c)
{
    const int ideal = bucket_bits(c->n_bound);
    return c->bucketed && c->hb >= ideal - 1 && c->hb <= ideal + 2;
}

// the most terms that the qubits allow
u64 all_keys(const sts_ctx *c) { return c->n_qubits < 64 ? 1ull << c->n_qubits : ~0ull; }

// the size bound after a gate of m qubits and the cut that follows it
u64 bound_after(const sts_ctx *c, int m)
{
    const u64 cb = sat_shl(c->n_bound, m);
    return std::min(c->K ? std::min<u64>(c->K, cb) : cb, c->cap);
}

// the kernel description's part that depends on the state's order: the
// bucket geometry, or the sort's bucket bits
void place_gate(const sts_ctx *c, GateArg *g, const int *qubits)
{
    if (use_tiny(c, g->m)) return; // any order will do
    if (use_buckets(c, g->m)) {
        const int hb = buckets_suit(c) ? c->hb : bucket_bits(c->n_bound);
        const int delta = std::min(std::max(bucket_bits(bound_after(c, g->m)) - hb, 0), 4);
        g->bkt = bkt_plan(hb, delta, g->m, qubits, c->prev_m, c->prev_q);
    } else {
        g->hb = sts_radix_bits(sort_shape(c)) * sort_passes(c); // the bucket bits the sort uses
    }
}

// put the state in bucket order unless it is (sorting by the bucket hash's
// top digits: one 11-bit pass while that is enough and the passes are short)
sts_status bucketize(sts_ctx *c)
{
    if (buckets_suit(c)) return STS_OK;
    const int hb = bucket_bits(c->n_bound);
    const int shape = hb <= 11 ? STS_RADIX_11x8 : STS_RADIX_8x16;
    const int bits = sts_radix_bits(shape);
    const int npass = (hb + bits - 1) / bits;
    const int tiles = (int)std::max<u64>(ceil_div(c->n_bound, sts_radix_tile(shape)), 1);
    const int a = (c->cur + 1) % 3, b = (c->cur + 2) % 3;
    int src = c->cur, dst = a;
    for (int p = 0; p < npass; ++p) {
        for (int what = 0; what < 3; ++what) {
            const int kind = what == 0 ? STS_K_RADIX_HIST : (what == 1 ? STS_K_RADIX_SCAN : STS_K_RADIX_PASS);
            STS_LAUNCH(c, kind, launch_radix(what, STS_SORT_BY_BUCKET, shape, c->prec, c->keys[src], c->amps[src],
                                             c->keys[dst], c->amps[dst], &c->ctl->cnt[src], &c->ctl->cnt[dst],
                                             nullptr, 64 - bits * npass + bits * p, c->rcount, c->rprefix, c->rtotal,
                                             c->tiles_cap, tiles, c->stream));
        }
        src = dst;
        dst = dst == a ? b : a;
    }
    STS_LAUNCH(c, STS_K_RADIX_SCAN,
               launch_bucket_bounds(c->keys[src], &c->ctl->cnt[src], c->n_bound, hb, c->bd[c->bdc], c->stream));
    c->cur = src;
    c->hb = hb;
    c->bucketed = true;
    return STS_OK;
}

// entries of a share's slab (log2): the side buffer over the shares, at least
// four entries per term of a share
int slab_shift(const sts_ctx *c)
{
    const u64 shares = 1ull << (c->gate.bkt.hb - 2);
    int sh = 0;
    while (sh < 12 && (shares << (sh + 1)) <= c->scap) ++sh;
    return sh;
}

int bucket_tiles(const sts_ctx *c) { return 1 << (c->gate.bkt.hb - STS_BKT_DIMS); }

// the passes that write the pending bucketed step's survivors to buffer dst
sts_status bucket_write(sts_ctx *c, PassBufs b, int dst, u64 bound)
{
    const int tiles = bucket_tiles(c);
    if (!b.emit_copies) { // else k_bkt_select has the offsets
        if (!b.whole)
            STS_LAUNCH(c, STS_K_GROUP_EXTRACT,
                       launch_bucket_pass(STS_BKT_COUNT, c->prec, c->gate.m, b, tiles, c->stream));
        STS_LAUNCH(c, STS_K_TILE_KEPT, launch_bucket_kept(b, tiles, c->stream));
        if (b.materialise && c->n_bound <= kSelectMax) b.emit_copies = 1; // a launch less
    }
    const bool copied = !b.emit_copies;
    if (copied)
        STS_LAUNCH(c, STS_K_GROUP_EMIT, launch_bucket_pass(STS_BKT_COPY, c->prec, c->gate.m, b, tiles, c->stream));
    STS_LAUNCH(c, copied ? STS_K_GROUP_EXTRACT : STS_K_GROUP_EMIT, launch_bucket_pass(STS_BKT_EMIT, c->prec, c->gate.m, b, tiles, c->stream));
    c->cur = dst;
    c->n_bound = bound;
    c->hb = c->gate.bkt.hb + c->gate.bkt.delta;
    c->bdc ^= 1;
    c->bucketed = true;
    c->bkt_pending = c->pending = false;
    c->prev_m = c->gate.m;
    for (int t = 0; t < c->gate.m; ++t) c->prev_q[t] = c->gate.q[t];
    return STS_OK;
}

// a one-launch step that may not fit the capacity takes the sorted passes
// instead, which can be counted first and refused
sts_status tiny_to_sorted(sts_ctx *c)
{
    int hb = 8, sorted = c->cur;
    c->gate.hb = sts_radix_bits(sort_shape(c)) * sort_passes(c);
    STS_TRY(c, launch_set_gate(c->gate, c->dgate, c->stream));
    c->gate_dev = c->dgate;
    c->bucketed = false;
    const sts_status st = sort_state(c, &c->dgate->notmask, &sorted, &hb);
    if (st != STS_OK) return st;
    c->cur = sorted;
    c->tiny_pending = false;
    return STS_OK;
}

// the pending one-launch step, its result in buffer dst
sts_status tiny_step(sts_ctx *c, PassBufs &b, int dst, u64 bound)
{
    STS_LAUNCH(c, STS_K_FINAL, launch_tiny(c->prec, c->gate, b, c->n_bound, c->stream));
    c->cur = dst;
    c->n_bound = bound;
    c->bucketed = false;
    c->tiny_pending = c->pending = false;
    return STS_OK;
}

// number of nonzero candidates of the pending gate (synchronises)
sts_status count_candidates(sts_ctx *c, u64 *count)
{
    PassBufs b = pass_bufs(c, c->cur, -1);
    if (c->bkt_pending) {
        b.whole = 1;
        STS_LAUNCH(c, STS_K_GROUP_HIST,
                   launch_bucket_pass(STS_BKT_HIST, c->prec, c->gate.m, b, bucket_tiles(c), c->stream));
        STS_LAUNCH(c, STS_K_PICK1, launch_pick1(b, 0, 1, 0, c->stream));
        const sts_status st = sync_ctl(c);
        if (st != STS_OK) return st;
        *count = c->hctl->cand_all;
        return STS_OK;
    }
    const bool tiled = use_tiles(c, c->gate.m);
    const int G = hist_groups(c->prec, c->n_bound, c->gate.m, tiled);
    STS_LAUNCH(c, STS_K_GROUP_HIST, launch_group_hist(c->prec, c->gate, b, G, tiled, c->stream));
    STS_LAUNCH(c, STS_K_PICK1, launch_pick1(b, G, 1, 0, c->stream));
    const sts_status st = sync_ctl(c);
    if (st != STS_OK) return st;
    *count = c->hctl->cand_all;
    return STS_OK;
}

// write out the pending gate's candidates without truncation
sts_status materialise(sts_ctx *c)
{
    if (!c->pending) return STS_OK;
    const u64 cb = sat_shl(c->n_bound, c->gate.m);
    u64 bound = cb;
    if (c->bkt_pending) STS_TRY(c, launch_set_gate(c->gate, c->dgate, c->stream));
    if (c->tiny_pending) {
        if (cb <= c->cap) {
            const int dst = (c->cur + 1) % 3;
            PassBufs b = pass_bufs(c, c->cur, dst);
            b.materialise = 1;
            return tiny_step(c, b, dst, cb);
        }
        const sts_status st = tiny_to_sorted(c);
        if (st != STS_OK) return st;
    }
    if (cb > c->cap) {
        u64 count = 0;
        const sts_status st = count_candidates(c, &count);
        if (st != STS_OK) return st;
        if (count > c->cap) {
            c->pending = c->bkt_pending = false; // drop the gate: the sorted input is the state before it
            return STS_E_CAPACITY;
        }
        bound = count;
    }
    const int dst = (c->cur + 1) % 3;
    PassBufs b = pass_bufs(c, c->cur, dst);
    b.materialise = 1;
    if (c->bkt_pending) {
        b.slab_shift = slab_shift(c);
        return bucket_write(c, b, dst, std::min(bound, c->cap));
    }
    if (use_tiles(c, c->gate.m)) {
        const int tt = (int)std::max<u64>(ceil_div(c->n_bound, 2048), 1);
        STS_LAUNCH(c, STS_K_GROUP_EXTRACT,
                   launch_group_extract_tiles(c->prec, c->gate, b, std::min(tt, 2048), c->stream));
        STS_LAUNCH(c, STS_K_TILE_KEPT, launch_tile_kept(b, tt, c->stream));
        STS_LAUNCH(c, STS_K_TILE_SCAN, launch_tile_scan(b, tt, c->stream));
        STS_LAUNCH(c, STS_K_GROUP_EMIT, launch_group_emit_tiles(c->prec, c->gate, b, tt, c->stream));
    } else {
        b.epoch = next_epoch(c);
        STS_LAUNCH(c, STS_K_GROUP_EMIT, launch_group_compact(c->prec, STS_KIND_EMIT, c->gate, b,
                                                             compact_tiles(c->n_bound, c->gate.m), c->stream));
    }
    c->cur = dst;
    c->n_bound = std::min(bound, c->cap);
    c->bucketed = false;
    c->pending = false;
    return STS_OK;
}

// the gate's kernel description (everything but the bucket bits hb, and
// for m >= 4 the device pointer to U); qubits and U already checked
void fill_gate(GateArg *g, int m, const int *qubits, const double *U)
{
    std::memset(g, 0, sizeof(*g));
    g->m = m;
    u64 mask = 0;
    for (int t = 0; t < m; ++t) {
        g->q[t] = qubits[t];
        mask |= 1ull << qubits[t];
    }
    g->notmask = ~mask;
    const int dim = 1 << m;
    if (m <= 3) {
        for (int i = 0; i < dim * dim; ++i) {
            g->ur[i] = U[2 * i];
            g->ui[i] = U[2 * i + 1];
            g->fr[i] = (float)U[2 * i]; // nearest-even
            g->fi[i] = (float)U[2 * i + 1];
        }
        for (int i = 0; i < dim; ++i) {
            u64 d = 0;
            for (int t = 0; t < m; ++t)
                if ((i >> t) & 1) d |= 1ull << qubits[t];
            g->dep[i] = d;
        }
    }
}

// STS_E_ARG unless qubits are m distinct qubits of the state and U is finite
sts_status check_gate(const sts_ctx *c, int m, const int *qubits, const double *U)
{
    if (!qubits || !U || m < 1 || m > STS_MAXM || m > c->n_qubits) return STS_E_ARG;
    u64 mask = 0;
    for (int t = 0; t < m; ++t) {
        if (qubits[t] < 0 || qubits[t] >= c->n_qubits) return STS_E_ARG;
        if (mask & (1ull << qubits[t])) return STS_E_ARG;
        mask |= 1ull << qubits[t];
    }
    for (int i = 0; i < 2 << (2 * m); ++i)
        if (!std::isfinite(U[i])) return STS_E_ARG;
    return STS_OK;
}

GateArg identity_gate()
{
    GateArg g;
    std::memset(&g, 0, sizeof(g));
    g.m = 0;
    g.notmask = ~0ull;
    return g;
}

sts_status check_live(sts_ctx *c)
{
    if (!c) return STS_E_ARG;
    if (c->poisoned) return STS_E_STATE;
    return STS_OK;
}

} // namespace

extern "C" {

sts_status sts_required_bytes(uint64_t cap_terms, int precision, size_t *bytes)
{
    if (!bytes || cap_terms == 0 || (precision != STS_C128 && precision != STS_C64)) return STS_E_ARG;
    if (cap_terms > (1ull << 36)) return STS_E_ARG;
    *bytes = (size_t)make_layout(cap_terms, precision).total;
    return STS_OK;
}

sts_status sts_init(sts_ctx **out, int n_qubits, uint64_t max_terms, double mass, int precision, void *hip_stream,
                    void *arena, size_t arena_bytes, uint64_t cap_terms)
{
    if (!out) return STS_E_ARG;
    *out = nullptr;
    if (n_qubits < 1 || n_qubits > 64) return STS_E_ARG;
    if (precision != STS_C128 && precision != STS_C64) return STS_E_ARG;
    if (!(mass == mass)) return STS_E_ARG; // NaN
    if (arena && arena_bytes == 0) return STS_E_ARG;
    if (cap_terms > (1ull << 36)) return STS_E_ARG;
    // n qubits have at most 2^n basis keys, so a larger K never cuts
    if (n_qubits < 64) max_terms = std::min<u64>(max_terms, 1ull << n_qubits);
    u64 cap = cap_terms;
    if (arena) {
        if (cap == 0) {
            // largest capacity whose layout fits the arena
            u64 lo = 1, hi = 1ull << 36;
            if (make_layout(1, precision).total > arena_bytes) return STS_E_NOMEM;
            while (lo < hi) {
                const u64 mid = lo + (hi - lo + 1) / 2;
                if (make_layout(mid, precision).total <= arena_bytes) lo = mid;
                else hi = mid - 1;
            }
            cap = lo;
        }
        if (make_layout(cap, precision).total > arena_bytes) return STS_E_NOMEM;
    } else if (cap == 0) {
        cap = std::max<u64>(max_terms, 1ull << 20);
    }
    if (max_terms > cap) return STS_E_CAPACITY;

    sts_ctx *c = new (std::nothrow) sts_ctx();
    if (!c) return STS_E_NOMEM;
    c->n_qubits = n_qubits;
    c->prec = precision;
    c->K = max_terms;
    c->p = (mass > 0.0 && mass < 1.0) ? mass : 0.0;
    c->stream = (hipStream_t)hip_stream;
    c->cap = cap;
    c->scap = side_capacity(cap);
    c->tiles_cap = ceil_div(cap, 2048) + 1;
    c->gtiles_cap = ceil_div(cap, STS_GTILE);
    const Layout L = make_layout(cap, precision);
    if (arena) {
        c->mem = (unsigned char *)arena;
    } else {
        void *p = nullptr;
        const hipError_t e = hipMalloc(&p, L.total);
        if (e != hipSuccess) {
            delete c;
            return e == hipErrorOutOfMemory ? STS_E_NOMEM : STS_E_HIP;
        }
        c->mem = (unsigned char *)p;
        c->own_mem = true;
    }
    bind_layout(c, L);

    hipError_t e = hipHostMalloc((void **)&c->hctl, sizeof(DevCtl), hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipHostMalloc((void **)&c->hU, kULen * (sizeof(double) + sizeof(float)), hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->u_event, hipEventDisableTiming);
    if (e != hipSuccess) {
        sts_free(c);
        return STS_E_HIP;
    }
    std::memset(c->hctl, 0, sizeof(DevCtl));
    c->hctl->K = c->K;
    c->hctl->p = c->p;
    c->hctl->scale = 1.0;
    c->hctl->frac = 1.0;
    c->hctl->e_pred = -1;
    // zero the bookkeeping regions (everything but the term buffers)
    e = hipMemsetAsync(c->mem + L.h1, 0, L.total - L.h1, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->ctl, c->hctl, sizeof(DevCtl), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = launch_init_state(precision, c->keys[0], c->amps[0], &c->ctl->cnt[0], c->stream);
    if (e == hipSuccess) e = launch_set_gate(identity_gate(), c->dgate_id, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        sts_free(c);
        return e == hipErrorOutOfMemory ? STS_E_NOMEM : STS_E_HIP;
    }
    c->cur = 0;
    c->n_bound = 1;
    *out = c;
    return STS_OK;
}

sts_status sts_apply_gate(sts_ctx *c, int m, const int *qubits, const double *U)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    st = check_gate(c, m, qubits, U);
    if (st != STS_OK) return st;
    st = materialise(c);
    if (st != STS_OK) return st;

    GateArg g;
    fill_gate(&g, m, qubits, U);
    const int dim = 1 << m;
    if (m > 3) {
        // the previous copy from the staging buffer must have finished
        if (c->u_event_live) STS_TRY(c, hipEventSynchronize(c->u_event));
        // the FP64 entries, then their FP32 roundings (nearest-even) right
        // after them: one copy
        const size_t nd = (size_t)2 * dim * dim;
        std::memcpy(c->hU, U, nd * sizeof(double));
        float *hf = reinterpret_cast<float *>(c->hU + nd);
        for (size_t i = 0; i < nd; ++i) hf[i] = (float)U[i];
        STS_TRY(c, hipMemcpyAsync(c->dU, c->hU, nd * (sizeof(double) + sizeof(float)), hipMemcpyHostToDevice,
                                  c->stream));
        STS_TRY(c, hipEventRecord(c->u_event, c->stream));
        c->u_event_live = true;
        g.uptr = c->dU;
        g.uptr_f = reinterpret_cast<const float *>(c->dU + nd);
    }
    int sorted = c->cur, hb = 8;
    place_gate(c, &g, qubits);
    if (use_tiny(c, m)) { // the whole step is the next call's one launch
        c->gate = g;
        c->pending = c->tiny_pending = true;
        return STS_OK;
    }
    c->gate_dev = c->dgate;
    if (use_buckets(c, m)) { // (the gate goes to the device with the next call's first kernel)
        st = bucketize(c);
        if (st != STS_OK) return st;
        c->gate = g;
        c->pending = c->bkt_pending = true;
        return STS_OK;
    }
    STS_TRY(c, launch_set_gate(g, c->dgate, c->stream));
    c->bucketed = false;
    st = sort_state(c, &c->dgate->notmask, &sorted, &hb);
    if (st != STS_OK) return st;
    c->cur = sorted;
    c->gate = g;
    c->pending = true;
    return STS_OK;
}

static sts_status truncate_buckets(sts_ctx *c)
{
    const u64 cb = sat_shl(c->n_bound, c->gate.m);
    const int out = (c->cur + 1) % 3;
    PassBufs b = pass_bufs(c, c->cur, out);
    const int m = c->gate.m, tiles = bucket_tiles(c);
    b.slab_shift = slab_shift(c);
    u64 nb = c->K ? std::min<u64>(c->K, cb) : cb;
    sts_status st = STS_OK;
    const bool out_risk = nb > c->cap; // a cut limited by p-mass alone may keep more than cap terms
    b.may_refuse = out_risk;
    if (out_risk) {
        st = save_ctl(c);
        if (st != STS_OK) return st;
    }
    const bool small = c->n_bound <= kSelectMax && tiles * 4 <= STS_SEL_SHARES;
    b.keep = 1;
    b.recover = 1;
    if (!small && c->p == 0.0 && (c->K == 0 || std::min(cb, all_keys(c)) <= c->K)) {
        // nothing can be cut: the histogram for the statistics, then the write
        b.whole = 1;
        STS_TRY(c, launch_set_gate(c->gate, c->dgate, c->stream));
        STS_LAUNCH(c, STS_K_GROUP_HIST, launch_bucket_pass(STS_BKT_HIST, c->prec, m, b, tiles, c->stream));
    } else if (small && c->n_bound > kSmallMax) {
        b.fine_window = 1;
        STS_LAUNCH(c, STS_K_SAMPLE, launch_bucket_pass(STS_BKT_SAMPLE, c->prec, m, b, tiles, c->stream, &c->gate));
        STS_LAUNCH(c, STS_K_GROUP_HIST, launch_bucket_pass(STS_BKT_MID, c->prec, m, b, tiles, c->stream));
        STS_LAUNCH(c, STS_K_FINAL, launch_bucket_pass(STS_BKT_SELECT_MID, c->prec, m, b, tiles, c->stream));
        b.emit_copies = 1;
    } else if (small) {
        STS_LAUNCH(c, STS_K_GROUP_HIST, launch_bucket_pass(STS_BKT_SMALL, c->prec, m, b, tiles, c->stream, &c->gate));
        STS_LAUNCH(c, STS_K_FINAL, launch_bucket_pass(STS_BKT_SELECT, c->prec, m, b, tiles, c->stream));
        b.emit_copies = 1;
    } else {
        // a window from a sample; the histogram pass and its pick run only
        // when it missed
        STS_LAUNCH(c, STS_K_SAMPLE, launch_bucket_pass(STS_BKT_SAMPLE, c->prec, m, b, tiles, c->stream, &c->gate));
        STS_LAUNCH(c, STS_K_GROUP_HIST, launch_bucket_pass(STS_BKT_WEIGH, c->prec, m, b, tiles, c->stream));
        STS_LAUNCH(c, STS_K_PICK1, launch_pick_window(b, bucket_weigh_groups(c->prec, m, tiles), c->stream));
        // (timed apart from the passes that do the work)
        STS_LAUNCH(c, STS_K_SIDE_HIST, launch_bucket_pass(STS_BKT_HIST, c->prec, m, b, tiles, c->stream));
        STS_LAUNCH(c, STS_K_GROUP_EXTRACT, launch_bucket_pass(STS_BKT_EXTRACT, c->prec, m, b, tiles, c->stream));
        const int sg =
            (int)std::min<u64>(std::max<u64>(ceil_div(std::min(cb, c->scap), 256), 1), STS_SIDE_GROUPS);
        STS_LAUNCH(c, STS_K_SIDE_EXTRACT, launch_side_extract(b, std::max(sg, (tiles + 3) / 4), c->stream));
        STS_LAUNCH(c, STS_K_FINAL, launch_final(b, c->stream));
    }
    if (out_risk) {
        st = sync_ctl(c);
        if (st != STS_OK) return st;
        const u64 L = c->hctl->keep_all ? c->hctl->n_cand : c->hctl->L;
        if (L > c->cap) return refuse_step(c);
        nb = L;
    }
    return bucket_write(c, b, out, nb);
}

sts_status sts_truncate(sts_ctx *c)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (c->pending && c->bkt_pending) return truncate_buckets(c);
    if (c->pending && c->tiny_pending) {
        const u64 cb = sat_shl(c->n_bound, c->gate.m);
        const u64 nb = c->K ? std::min<u64>(c->K, cb) : cb;
        if (nb <= c->cap) {
            const int out = (c->cur + 1) % 3;
            PassBufs b = pass_bufs(c, c->cur, out);
            return tiny_step(c, b, out, nb);
        }
        st = tiny_to_sorted(c); // a cut limited by p-mass alone may keep more than cap terms
        if (st != STS_OK) return st;
    }
    if (!c->pending) {
        c->gate = identity_gate();
        c->gate_dev = c->dgate_id;
        c->pending = true;
    }
    const u64 cb = sat_shl(c->n_bound, c->gate.m);
    const int out = (c->cur + 1) % 3;
    PassBufs b = pass_bufs(c, c->cur, out);
    const bool tiled = use_tiles(c, c->gate.m);
    const int G = hist_groups(c->prec, c->n_bound, c->gate.m, tiled);
    const int tiles = compact_tiles(c->n_bound, c->gate.m);
    const int tt = (int)std::max<u64>(ceil_div(c->n_bound, 2048), 1);
    u64 nb = c->K ? std::min<u64>(c->K, cb) : cb;
    // two ways a step may not fit, both found before anything is written:
    // untiled passes (4- and 5-qubit gates on a large state) copy the cut
    // exponent's candidates to the side buffer in one dense run, which may
    // exceed it; a cut limited by p-mass alone may keep more than cap terms
    const bool side_risk = !tiled && cb > c->scap;
    const bool out_risk = nb > c->cap;
    if (side_risk || out_risk) {
        st = save_ctl(c);
        if (st != STS_OK) return st;
    }
    // large states: estimate this step's cut on a sample of tiles first, so
    // that the histogram pass copies a narrow window around it
    if (tiled && c->gate.m >= 1 && c->gate.m <= 4 && c->n_bound >= STS_SAMPLE_MIN)
        STS_LAUNCH(c, STS_K_SAMPLE, launch_group_sample(c->prec, c->gate, b, c->stream));
    b.predict = tiled ? 1 : 0; // the histogram pass also extracts the predicted window
    // and keeps the candidates above it, so that a step whose cut falls in
    // the window writes its survivors without running the gate again
    b.copy = tiled ? 1 : 0;
    STS_LAUNCH(c, STS_K_GROUP_HIST, launch_group_hist(c->prec, c->gate, b, G, tiled, c->stream));
    b.predict = 0;
    STS_LAUNCH(c, STS_K_PICK1, launch_pick1(b, G, 0, tiled ? 1 : 0, c->stream));
    if (side_risk) {
        st = sync_ctl(c);
        if (st != STS_OK) return st;
        if (!c->hctl->keep_all && c->hctl->sub_count > c->scap) return refuse_step(c);
    }
    if (tiled) {
        // as many workgroups as the histogram pass keeps resident: one round
        // of launches when the window held the cut and every one exits
        STS_LAUNCH(c, STS_K_GROUP_EXTRACT,
                   launch_group_extract_tiles(c->prec, c->gate, b, std::min(tt, G), c->stream));
    } else {
        b.epoch = next_epoch(c);
        STS_LAUNCH(c, STS_K_GROUP_EXTRACT,
                   launch_group_compact(c->prec, STS_KIND_EXTRACT, c->gate, b, tiles, c->stream));
    }
    // the side passes stream the side buffer; 128 workgroups keep it moving,
    // and more would only queue more atomics on the shared bins and the
    // last-workgroup counter
    const int sg = (int)std::min<u64>(std::max<u64>(ceil_div(std::min(cb, c->scap), 256), 1), STS_SIDE_GROUPS);
    STS_LAUNCH(c, STS_K_SIDE_HIST, launch_side_hist(b, c->h2, sg, c->stream));
    // the extraction keeps no per-workgroup state: one wave per tile keeps
    // every tile's loads in flight at once
    STS_LAUNCH(c, STS_K_SIDE_EXTRACT, launch_side_extract(b, tiled ? std::max(sg, (tt + 3) / 4) : sg, c->stream));
    STS_LAUNCH(c, STS_K_FINAL, launch_final(b, c->stream));
    if (out_risk) {
        // only p-mass limits this cut: learn its size before writing
        st = sync_ctl(c);
        if (st != STS_OK) return st;
        const u64 L = c->hctl->keep_all ? c->hctl->n_cand : c->hctl->L;
        if (L > c->cap) return refuse_step(c);
        nb = L;
    }
    if (tiled) {
        STS_LAUNCH(c, STS_K_TILE_KEPT, launch_tile_kept(b, tt, c->stream));
        STS_LAUNCH(c, STS_K_TILE_SCAN, launch_tile_scan(b, tt, c->stream));
        STS_LAUNCH(c, STS_K_GROUP_EMIT, launch_group_emit_tiles(c->prec, c->gate, b, tt, c->stream));
    } else {
        b.epoch = next_epoch(c);
        STS_LAUNCH(c, STS_K_GROUP_EMIT, launch_group_compact(c->prec, STS_KIND_EMIT, c->gate, b, tiles, c->stream));
    }
    c->cur = out;
    c->n_bound = nb;
    c->bucketed = false;
    c->pending = false;
    return STS_OK;
}

sts_status sts_set_sort_shape(sts_ctx *c, int small_log2, int shape)
{
    static_assert(STS_SORT_8x16 == STS_RADIX_8x16 && STS_SORT_8x8 == STS_RADIX_8x8 &&
                      STS_SORT_11x16 == STS_RADIX_11x16 && STS_SORT_11x8 == STS_RADIX_11x8,
                  "public and internal sort shapes agree");
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (small_log2 < 0 || small_log2 > 40 || shape < 0 || shape >= STS_RADIX_SHAPES) return STS_E_ARG;
    if (c->pending) return STS_E_STATE; // the pending gate's sort already ran with the old shape
    c->radix_small_log2 = small_log2;
    c->radix_small_shape = shape;
    return STS_OK;
}

sts_status sts_peak(sts_ctx *c, uint64_t *key, double *prob)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (!key || !prob) return STS_E_ARG;
    st = materialise(c);
    if (st != STS_OK) return st;
    const GateArg g = identity_gate();
    PassBufs b = pass_bufs(c, c->cur, -1);
    b.gate = c->dgate_id;
    const int G = hist_groups(c->prec, c->n_bound, 0, true);
    STS_LAUNCH(c, STS_K_GROUP_HIST, launch_group_hist(c->prec, g, b, G, true, c->stream));
    STS_LAUNCH(c, STS_K_PICK1, launch_pick1(b, G, 1, 0, c->stream));
    st = sync_ctl(c);
    if (st != STS_OK) return st;
    if (c->hctl->cnt[c->cur] == 0) return STS_E_STATE;
    *key = c->hctl->peak_key;
    *prob = c->hctl->peak_w / c->hctl->peak_W;
    return STS_OK;
}

sts_status sts_num_terms(sts_ctx *c, uint64_t *n)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (!n) return STS_E_ARG;
    st = materialise(c);
    if (st != STS_OK) return st;
    st = sync_ctl(c);
    if (st != STS_OK) return st;
    *n = c->hctl->cnt[c->cur];
    c->n_bound = *n;
    return STS_OK;
}

sts_status sts_read_terms(sts_ctx *c, uint64_t cap, uint64_t *keys, double *amps, uint64_t *n)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (!n || (cap && (!keys || !amps))) return STS_E_ARG;
    st = sts_num_terms(c, n);
    if (st != STS_OK) return st;
    const u64 cnt = *n;
    if (cnt > cap) return STS_E_CAPACITY;
    if (cnt == 0) return STS_OK;
    if (on_host(c, cnt)) return read_small(c, cnt, keys, amps);
    // sorted by key on the device, between the two free term buffers
    u64 *k = c->keys[c->cur];
    void *a = c->amps[c->cur];
    st = sort_by_key(c, cnt, c->prec, &k, &a, {c->keys[(c->cur + 1) % 3], c->keys[(c->cur + 2) % 3]},
                     {c->amps[(c->cur + 1) % 3], c->amps[(c->cur + 2) % 3]}, &c->ctl->cnt[c->cur]);
    if (st != STS_OK) return st;
    const void *wide = a;
    if (c->prec == STS_C64) { // the side buffer has room for the FP64 pairs
        STS_TRY(c, launch_widen((const float2 *)a, (double2 *)c->side_amp, cnt, c->stream));
        wide = c->side_amp;
    }
    STS_TRY(c, hipMemcpyAsync(keys, k, cnt * 8, hipMemcpyDeviceToHost, c->stream));
    STS_TRY(c, hipMemcpyAsync(amps, wide, cnt * 16, hipMemcpyDeviceToHost, c->stream));
    STS_TRY(c, hipStreamSynchronize(c->stream));
    return STS_OK;
}

sts_status sts_load_terms(sts_ctx *c, uint64_t n, const uint64_t *keys, const double *amps)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (n && (!keys || !amps)) return STS_E_ARG;
    if (n > c->cap) return STS_E_CAPACITY;
    const u64 lim = c->n_qubits == 64 ? ~0ull : ((1ull << c->n_qubits) - 1);
    const int dst = (c->cur + 1) % 3; // a free buffer: refused terms change nothing
    u32 most = 0;
    if (n && on_host(c, n)) {
        st = load_small(c, n, keys, amps, lim, dst, &most);
        if (st != STS_OK) return st;
    } else if (n) {
        // checked on the device: range and finiteness, then (sorted in the
        // side buffer) that no key comes twice
        double *wide = c->prec == STS_C128 ? (double *)c->amps[dst] : (double *)c->side_amp;
        STS_TRY(c, hipMemcpyAsync(c->keys[dst], keys, n * 8, hipMemcpyHostToDevice, c->stream));
        STS_TRY(c, hipMemcpyAsync(wide, amps, n * 16, hipMemcpyHostToDevice, c->stream));
        u64 *counts = c->cap <= kBucketMax ? (u64 *)c->bd[c->bdc ^ 1] : nullptr; // (the next bucketed step's table)
        STS_TRY(c, launch_load_check(c->prec, c->keys[dst], wide, n, lim, (float2 *)c->amps[dst], bucket_bits(n), counts,
                                     c->ctl, c->stream));
        STS_TRY(c, launch_set_n(&c->ctl->cnt[dst], n, c->stream));
        u64 *k = c->keys[dst];
        void *w = c->keys[dst]; // moved along with the keys, not used
        st = sort_by_key(c, n, STS_C64, &k, &w, {c->side_key, c->side_key + c->cap}, {c->side_w, c->side_w + c->cap},
                         &c->ctl->cnt[dst]);
        if (st != STS_OK) return st;
        STS_TRY(c, launch_load_unique(k, n, bucket_bits(n), counts, c->ctl, c->stream));
        st = sync_ctl(c); // also: the caller's arrays have been read
        if (st != STS_OK) return st;
        if (c->hctl->load_flags) {
            STS_TRY(c, hipMemsetAsync(&c->ctl->load_flags, 0, sizeof(u32), c->stream));
            return STS_E_ARG;
        }
        most = c->hctl->load_most;
    }
    // the state is replaced: any pending gate is dropped
    c->pending = c->bkt_pending = c->tiny_pending = false;
    c->bucketed = false;
    c->crowded = most >= kCrowded;
    c->cur = dst;
    STS_TRY(c, launch_set_n(&c->ctl->cnt[c->cur], n, c->stream));
    c->n_bound = n;
    return STS_OK;
}

sts_status sts_stats(sts_ctx *c, double *W, double *kept_fraction, double *log10_cum_kept, uint64_t *last_candidates)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    st = sync_ctl(c);
    if (st != STS_OK) return st;
    if (W) *W = c->hctl->W;
    if (kept_fraction) *kept_fraction = c->hctl->frac;
    if (log10_cum_kept) *log10_cum_kept = c->hctl->log10_cum;
    if (last_candidates) *last_candidates = c->hctl->n_cand;
    return STS_OK;
}

sts_status sts_counters(sts_ctx *c, uint64_t *gate_steps, uint64_t *term_updates, uint64_t *candidates)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    st = sync_ctl(c);
    if (st != STS_OK) return st;
    if (gate_steps) *gate_steps = c->hctl->tot_steps;
    if (term_updates) *term_updates = c->hctl->tot_updates;
    if (candidates) *candidates = c->hctl->tot_cand;
    return STS_OK;
}

sts_status sts_profile(sts_ctx *c, int enable)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    c->prof = enable != 0;
    return STS_OK;
}

sts_status sts_kernel_time(sts_ctx *c, int kind, int reset, double *total_ms, uint64_t *launches)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    if (kind < 0 || kind >= STS_K_COUNT) return STS_E_ARG;
    STS_TRY(c, hipStreamSynchronize(c->stream));
    prof_collect(c);
    if (total_ms) *total_ms = c->prof_ms[kind];
    if (launches) *launches = c->prof_n[kind];
    if (reset) {
        for (int k = 0; k < STS_K_COUNT; ++k) {
            c->prof_ms[k] = 0;
            c->prof_n[k] = 0;
        }
    }
    return STS_OK;
}

sts_status sts_step_static(int n_qubits, uint64_t max_terms, double mass, int precision, void *hip_stream, int m,
                           const int *qubits, const double *U, const uint64_t *keys_in, const void *amps_in,
                           uint64_t n_in, uint64_t *keys_out, void *amps_out, uint64_t *n_out, double *stats)
{
    if (n_qubits < 1 || n_qubits > 64 || (precision != STS_C128 && precision != STS_C64)) return STS_E_ARG;
    if (!(mass == mass) || !qubits || !U || m < 1 || m > 3 || m > n_qubits) return STS_E_ARG;
    if ((n_in && (!keys_in || !amps_in)) || !keys_out || !amps_out || !n_out) return STS_E_ARG;
    if (n_qubits < 64) max_terms = std::min<u64>(max_terms, 1ull << n_qubits);
    if (max_terms == 0) return STS_E_ARG; // top-k bounds the result and the caller's output arrays
    if (max_terms > STS_STATIC_MAX_TERMS || n_in > STS_STATIC_MAX_TERMS) return STS_E_CAPACITY;
    const Layout L = make_layout(STS_STATIC_MAX_TERMS, precision);
    if (L.total > kStaticBytes) return STS_E_CAPACITY;
    void *base = nullptr;
    if (static_scratch(&base) != hipSuccess) return STS_E_HIP;

    // a context on the stack over the static array: with gates of at most 3
    // qubits and top-k within the capacity, the gate step never synchronises,
    // never allocates and is never refused
    sts_ctx c;
    c.n_qubits = n_qubits;
    c.prec = precision;
    c.K = max_terms;
    c.p = (mass > 0.0 && mass < 1.0) ? mass : 0.0;
    c.stream = (hipStream_t)hip_stream;
    c.cap = STS_STATIC_MAX_TERMS;
    c.scap = side_capacity(c.cap);
    c.tiles_cap = ceil_div(c.cap, 2048) + 1;
    c.gtiles_cap = ceil_div(c.cap, STS_GTILE);
    c.mem = (unsigned char *)base;
    bind_layout(&c, L);
    // the array keeps the last call's contents: every counter, histogram and
    // look-back word starts from zero again, and the control block anew
    STS_TRY(&c, launch_fill_zero((u64 *)(c.mem + L.h1), (L.total - L.h1) / 8, c.stream));
    STS_TRY(&c, launch_ctl_begin(c.ctl, c.K, c.p, n_in, c.stream));
    STS_TRY(&c, launch_set_gate(identity_gate(), c.dgate_id, c.stream));
    const u64 asz = precision == STS_C128 ? 16 : 8;
    if (n_in) {
        STS_TRY(&c, hipMemcpyAsync(c.keys[0], keys_in, n_in * 8, hipMemcpyDeviceToDevice, c.stream));
        STS_TRY(&c, hipMemcpyAsync(c.amps[0], amps_in, n_in * asz, hipMemcpyDeviceToDevice, c.stream));
    }
    c.cur = 0;
    c.n_bound = n_in;
    c.one_step = true;
    sts_status st = sts_apply_gate(&c, m, qubits, U);
    if (st != STS_OK) return st;
    st = sts_truncate(&c);
    if (st != STS_OK) return st;
    STS_TRY(&c, launch_terms_out(c.keys[c.cur], c.amps[c.cur], (int)asz, c.ctl, c.cur, (u64 *)keys_out, amps_out,
                                 max_terms, (u64 *)n_out, stats, c.stream));
    return STS_OK;
}

void sts_free(sts_ctx *c)
{
    if (!c) return;
    if (c->stream || c->mem) (void)hipStreamSynchronize(c->stream);
    for (auto &m : c->marks) {
        (void)hipEventDestroy(m.a);
        (void)hipEventDestroy(m.b);
    }
    for (auto e : c->pool) (void)hipEventDestroy(e);
    if (c->own_mem && c->mem) (void)hipFree(c->mem);
    if (c->hctl) (void)hipHostFree(c->hctl);
    if (c->hU) (void)hipHostFree(c->hU);
    if (c->u_event) (void)hipEventDestroy(c->u_event);
    delete c;
}

const char *sts_strerror(sts_status s)
{
    switch (s) {
    case STS_OK: return "ok";
    case STS_E_ARG: return "invalid argument";
    case STS_E_NOMEM: return "device allocation failed";
    case STS_E_CAPACITY: return "result exceeds the context's capacity";
    case STS_E_HIP: return "HIP runtime error";
    case STS_E_STATE: return "context poisoned or call out of order";
    }
    return "unknown status";
}

} // extern "C"

// ---------------------------------------------------------------------------
// Replayed gate steps (batch runner). A truncated step of up to 3 qubits
// launches the same kernels with the same grids whenever the context starts
// it from the same term buffer with the same size bound: every size the
// kernels use is read from device memory, and the gate itself from the
// context's device copy, written by the one launch that is given it: the
// step's first kernel, or k_set_gate. Such a step is captured into a HIP graph
// once and afterwards replayed with only that launch's argument changed to the
// new gate.
// ---------------------------------------------------------------------------
struct StepGraph {
    int m, cur;
    u64 nb;
    hipGraph_t graph;
    hipGraphExec_t exec;
    hipGraphNode_t set_node;
    int cur_after;
    u64 nb_after;
    bool bucketed;       // the state's order before the step, and after
    int hb, bdc;
    bool bucketed_after;
    int hb_after, bdc_after;
};

struct StepGraphs {
    std::vector<StepGraph> v;
    u64 last_nb = ~0ull;
    u64 replays = 0, captures = 0;
};

StepGraphs *step_graphs_new() { return new (std::nothrow) StepGraphs(); }

void step_graphs_free(StepGraphs *gs)
{
    if (!gs) return;
    for (auto &e : gs->v) {
        if (e.exec) (void)hipGraphExecDestroy(e.exec);
        if (e.graph) (void)hipGraphDestroy(e.graph);
    }
    delete gs;
}

void step_graphs_counts(const StepGraphs *gs, u64 *captures, u64 *replays)
{
    *captures = gs ? gs->captures : 0;
    *replays = gs ? gs->replays : 0;
}

sts_status step_replayed(sts_ctx *c, StepGraphs *gs, int m, const int *qubits, const double *U)
{
    sts_status st = check_live(c);
    if (st != STS_OK) return st;
    st = check_gate(c, m, qubits, U);
    if (st != STS_OK) return st;
    // a steady size bound (as the previous step's) and a step that never
    // synchronises: gates of up to 3 qubits, top-k within the capacity
    const bool steady = c->n_bound == gs->last_nb;
    gs->last_nb = c->n_bound;
    if (!steady || c->pending || c->prof || m > 3 || c->K == 0 || c->K > c->cap) {
        st = sts_apply_gate(c, m, qubits, U);
        if (st == STS_OK) st = sts_truncate(c);
        return st;
    }
    StepGraph *hit = nullptr;
    for (auto &e : gs->v)
        if (e.m == m && e.cur == c->cur && e.nb == c->n_bound && e.bucketed == c->bucketed &&
            e.bdc == c->bdc && (!e.bucketed || e.hb == c->hb))
            hit = &e;
    if (!hit) {
        StepGraph e{};
        e.m = m;
        e.cur = c->cur;
        e.nb = c->n_bound;
        e.bucketed = c->bucketed;
        e.hb = c->hb;
        e.bdc = c->bdc;
        STS_TRY(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
        st = sts_apply_gate(c, m, qubits, U);
        if (st == STS_OK) st = sts_truncate(c);
        hipGraph_t graph = nullptr;
        const hipError_t ee = hipStreamEndCapture(c->stream, &graph);
        if (st != STS_OK || ee != hipSuccess || !graph) {
            if (graph) (void)hipGraphDestroy(graph);
            c->poisoned = true; // the step was recorded, not run
            return st != STS_OK ? st : STS_E_HIP;
        }
        e.graph = graph;
        e.cur_after = c->cur;
        e.nb_after = c->n_bound;
        e.bucketed_after = c->bucketed;
        e.hb_after = c->hb;
        e.bdc_after = c->bdc;
        // the one launch that is given the gate
        size_t nn = 0;
        hipError_t he = hipGraphGetNodes(graph, nullptr, &nn);
        std::vector<hipGraphNode_t> nodes(nn);
        if (he == hipSuccess) he = hipGraphGetNodes(graph, nodes.data(), &nn);
        for (size_t i = 0; he == hipSuccess && i < nn; ++i) {
            hipGraphNodeType t;
            if (hipGraphNodeGetType(nodes[i], &t) != hipSuccess || t != hipGraphNodeTypeKernel) continue;
            hipKernelNodeParams p{};
            if (hipGraphKernelNodeGetParams(nodes[i], &p) == hipSuccess &&
                (p.func == set_gate_kernel() ||
                 (m <= 2 && (is_tiny_kernel(p.func, c->prec, m) ||
                             p.func == bucket_first_kernel(STS_BKT_SMALL, c->prec, m) ||
                             p.func == bucket_first_kernel(STS_BKT_SAMPLE, c->prec, m)))))
                e.set_node = nodes[i];
        }
        if (he == hipSuccess && !e.set_node) he = hipErrorNotFound;
        if (he == hipSuccess) he = hipGraphInstantiate(&e.exec, graph, nullptr, nullptr, 0);
        if (he == hipSuccess) he = hipGraphLaunch(e.exec, c->stream);
        if (he != hipSuccess) {
            if (e.exec) (void)hipGraphExecDestroy(e.exec);
            (void)hipGraphDestroy(graph);
            return fail_hip(c, he);
        }
        gs->v.push_back(e);
        gs->captures += 1;
        return STS_OK;
    }
    // replay with the new gate: the same bucket bits (same size bound)
    GateArg g;
    fill_gate(&g, m, qubits, U);
    place_gate(c, &g, qubits);
    if (use_buckets(c, m)) {
        c->prev_m = m;
        for (int t = 0; t < m; ++t) c->prev_q[t] = qubits[t];
    }
    // the node's first argument is the gate; the others stay
    hipKernelNodeParams p{};
    STS_TRY(c, hipGraphKernelNodeGetParams(hit->set_node, &p));
    void *args[2] = {&g, p.kernelParams[1]};
    p.kernelParams = args;
    p.extra = nullptr;
    STS_TRY(c, hipGraphExecKernelNodeSetParams(hit->exec, hit->set_node, &p));
    STS_TRY(c, hipGraphLaunch(hit->exec, c->stream));
    c->cur = hit->cur_after;
    c->n_bound = hit->nb_after;
    c->bucketed = hit->bucketed_after;
    c->hb = hit->hb_after;
    c->bdc = hit->bdc_after;
    c->gate = g;
    c->gate_dev = c->dgate;
    c->pending = false;
    gs->replays += 1;
    return STS_OK;
}
