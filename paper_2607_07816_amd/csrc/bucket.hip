// bucket.hip - bucketed and one-launch gate steps: dispatch by precision, the survivor
// counts and offsets, and the bucket table of a freshly ordered state.
#include <algorithm>

#include "kernels.h"

hipError_t bucket_c128_pass(int kind, int m, const PassBufs &b, int tiles, hipStream_t s, const GateArg *first);
const void *bucket_c128_first(int kind, int m);
hipError_t bucket_c64_pass(int kind, int m, const PassBufs &b, int tiles, hipStream_t s, const GateArg *first);
const void *bucket_c64_first(int kind, int m);
hipError_t tiny_c128(const GateArg &g, const PassBufs &b, u64 n_bound, hipStream_t s);
hipError_t tiny_c64(const GateArg &g, const PassBufs &b, u64 n_bound, hipStream_t s);
const void *tiny_c128_kernel(int m, int size);
const void *tiny_c64_kernel(int m, int size);
int bucket_c128_groups(int m, int tiles);
int bucket_c64_groups(int m, int tiles);

namespace {

constexpr int KT = 256;

// The survivors of every share and the output offset of every tile. When the
// window held the cut, a share's survivors are its entries above the window
// and those of the window ranked at or above the threshold term (16 lanes per
// share, a wave per tile); when nothing is cut, all its candidates; otherwise
// the counting pass has them. A workgroup has STS_BKT_CHUNK tiles, whose
// offsets are relative to the chunk's base; the last workgroup scans the
// chunks' sums. Bound by the round trips to memory (a count, then a few window
// entries): a wave's eight tiles are loaded together, 24 us at 2^24 complex64
// terms, where two tiles one after the other, keys included, took 31.
__global__ void __launch_bounds__(KT) k_bkt_kept(PassBufs b)
{
    __shared__ u32 s_flag;
    __shared__ u32 s_tile[STS_BKT_CHUNK];
    __shared__ u64 s_scratch[KT / 64];
    constexpr int UN = 4;
    DevCtl *ctl = b.ctl;
    const u32 ntiles = 1u << (b.gate->bkt.hb - STS_BKT_DIMS);
    const u64 thr_w = ctl->thr_wbits, thr_k = ctl->thr_key;
    const int shift = ctl->side_slab_shift;
    const bool all = !b.materialise && ctl->keep_all, hit = !b.materialise && !ctl->keep_all && ctl->pred_hit;
    const u32 lane = (u32)sts_lane(), sub = lane >> 4, l16 = lane & 15u;
    const u32 t0 = blockIdx.x * STS_BKT_CHUNK;
    // a wave's tiles at a time, their loads in flight together
    constexpr u32 PW = STS_BKT_CHUNK / (KT / 64);
    const u32 k0 = threadIdx.x >> 6;
    u32 c[PW], ns[PW];
#pragma unroll
    for (u32 q = 0; q < PW; ++q) {
        const u32 tile = t0 + k0 + q * (KT / 64), sl = (tile << 2) + sub;
        const bool in = tile < ntiles;
        ns[q] = in && hit ? b.t_side[sl] : 0u;
        c[q] = !in ? 0u : hit ? (l16 == 0 ? b.t_above[sl] : 0u) : all ? b.w_all[sl] : b.w_kept[sl];
    }
    if (hit) {
        u64 w[PW][UN];
#pragma unroll
        for (u32 q = 0; q < PW; ++q) {
            const u64 base = (u64)(((t0 + k0 + q * (KT / 64)) << 2) + sub) << shift;
#pragma unroll
            for (int r = 0; r < UN; ++r) {
                const u32 i = l16 + 16u * (u32)r;
                w[q][r] = i < ns[q] ? b.side_w[base + i] : 0ull;
            }
        }
#pragma unroll
        for (u32 q = 0; q < PW; ++q) {
            const u64 base = (u64)(((t0 + k0 + q * (KT / 64)) << 2) + sub) << shift;
            // (the key decides between equal weights only, and is read for those)
            auto count = [&](u32 i, u64 x) {
                if (i < ns[q] && (x > thr_w || (x == thr_w && b.side_key[base + i] <= thr_k))) ++c[q];
            };
#pragma unroll
            for (int r = 0; r < UN; ++r) count(l16 + 16u * (u32)r, w[q][r]);
            for (u32 i = l16 + 16u * UN; i < ns[q]; i += 16) count(i, b.side_w[base + i]);
#pragma unroll
            for (int d = 8; d > 0; d >>= 1) c[q] += __shfl_xor(c[q], d, 64);
        }
    }
#pragma unroll
    for (u32 q = 0; q < PW; ++q) {
        const u32 tile = t0 + k0 + q * (KT / 64), sl = (tile << 2) + sub;
        if (tile < ntiles && l16 == 0 && (hit || all)) b.w_kept[sl] = c[q];
        c[q] += __shfl_xor(c[q], 16, 64);
        c[q] += __shfl_xor(c[q], 32, 64);
        if (lane == 0) s_tile[k0 + q * (KT / 64)] = c[q];
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        static_assert(STS_BKT_CHUNK <= 64, "one lane per tile");
        const u32 c = lane < STS_BKT_CHUNK ? s_tile[lane] : 0u;
        const u32 inc = wave_incl_scan(c);
        if (lane < STS_BKT_CHUNK && t0 + lane < ntiles) b.t_off[t0 + lane] = inc - c;
        if (lane == 63) st_agent(&b.t_base[blockIdx.x], (u64)inc);
    }
    if (!sts_last_block(&ctl->done[3], &s_flag)) return;
    u64 carry = 0;
    constexpr u32 PT = 8; // chunks of a thread at a time
    for (u32 i0 = 0; i0 < gridDim.x; i0 += KT * PT) {
        const u32 i = i0 + threadIdx.x * PT;
        u64 v[PT], sum = 0;
#pragma unroll
        for (u32 q = 0; q < PT; ++q) v[q] = i + q < gridDim.x ? ld_agent(&b.t_base[i + q]) : 0ull;
#pragma unroll
        for (u32 q = 0; q < PT; ++q) sum += v[q];
        u64 total;
        u64 run = block_excl_scan<u64, KT>(sum, s_scratch, &total) + carry;
#pragma unroll
        for (u32 q = 0; q < PT; ++q) {
            if (i + q < gridDim.x) st_agent(&b.t_base[i + q], run);
            run += v[q];
        }
        carry += total;
    }
    if (threadIdx.x == 0) {
        *b.n_out = carry;
        if (b.materialise) { // (the count has put the new terms into the slabs)
            ctl->slab_all = !ctl->w_over;
            ctl->w_over = 0;
        }
        if (carry > b.out_cap) atomicOr(&ctl->flags, STS_F_OUT_OVERFLOW);
    }
}

// bd[b] = (first, one past the last) term of bucket b; cleared before
__global__ void __launch_bounds__(256) k_bkt_bounds(const u64 *__restrict__ keys, const u64 *n_in, int hb, uint2 *bd)
{
    const u64 n = *n_in;
    const auto bucket = [&](u64 key) { // the top hb bits of the hash
        u32 v = 0;
        for (int i = 0; i < hb; ++i) v |= sts_parity(key, k_lin_masks[32 - hb + i]) << i;
        return v;
    };
    for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) {
        const u32 b1 = bucket(keys[i]);
        const bool first = i == 0 || bucket(keys[i - 1]) != b1;
        const bool last = i + 1 == n || bucket(keys[i + 1]) != b1;
        if (first) bd[b1].x = (u32)i;
        if (last) bd[b1].y = (u32)i + 1;
    }
}

} // namespace

int bucket_weigh_groups(int prec, int m, int tiles)
{
    return prec == 0 ? bucket_c128_groups(m, tiles) : bucket_c64_groups(m, tiles);
}

hipError_t launch_tiny(int prec, const GateArg &g, const PassBufs &b, u64 n_bound, hipStream_t s)
{
    return prec == 0 ? tiny_c128(g, b, n_bound, s) : tiny_c64(g, b, n_bound, s);
}

bool is_tiny_kernel(const void *func, int prec, int m)
{
    for (int size = 0; size < 3; ++size)
        if (func == (prec == 0 ? tiny_c128_kernel(m, size) : tiny_c64_kernel(m, size))) return true;
    return false;
}

hipError_t launch_bucket_pass(int kind, int prec, int m, const PassBufs &b, int tiles, hipStream_t s,
                              const GateArg *first)
{
    return prec == 0 ? bucket_c128_pass(kind, m, b, tiles, s, first) : bucket_c64_pass(kind, m, b, tiles, s, first);
}

const void *bucket_first_kernel(int kind, int prec, int m)
{
    return prec == 0 ? bucket_c128_first(kind, m) : bucket_c64_first(kind, m);
}

hipError_t launch_bucket_kept(const PassBufs &b, int tiles, hipStream_t s)
{
    const int grid = std::max(1, (tiles + STS_BKT_CHUNK - 1) / STS_BKT_CHUNK);
    hipLaunchKernelGGL(k_bkt_kept, dim3(grid), dim3(KT), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_bucket_bounds(const u64 *keys, const u64 *n_in, u64 n_bound, int hb, uint2 *bd, hipStream_t s)
{
    hipError_t e = launch_fill_zero(reinterpret_cast<u64 *>(bd), 1ull << hb, s);
    if (e != hipSuccess) return e;
    const u64 grid = std::max<u64>(1, std::min<u64>((n_bound + 255) / 256, 4096));
    hipLaunchKernelGGL(k_bkt_bounds, dim3((unsigned)grid), dim3(256), 0, s, keys, n_in, hb, bd);
    return hipGetLastError();
}
