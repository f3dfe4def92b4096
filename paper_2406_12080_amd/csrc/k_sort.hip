// Stable LSD radix sort of (uint32 key, uint32 value) pairs, 8-bit digits,
// LDS-staged, over one or more segments (one per view), each sorted in place
// on its own.  A fixed grid of blocks each owns one contiguous chunk of a
// segment (the element count is a device value, so the launches can be
// captured in a graph):
//   plan    : (once per sort) every segment's chunk size, blocks and first
//             block; the per-pass digit totals cleared
//   hist    : per-block digit histogram -> hist[segment][digit][block], and
//             the segment's digit totals
//   rowscan : one wave per (segment, digit): its first output slot (from the
//             totals of the lower digits) and the exclusive scan over the
//             segment's blocks, in place
//   scatter : each block walks its chunk in tiles, ranks keys stably inside
//             the tile (64-lane digit match from 8 ballots, per-wave running
//             counts in LDS), regroups the tile by digit in LDS, and writes
//             runs of equal digits contiguously.
// Ranking order inside a tile is (wave, item, lane) = input order, so equal
// keys keep their input order.
//
// Bounds: at 30M-90M elements the scatter is HBM-bound by partial lines (a
// digit's run in a tile of 4096 keys averages 64 B per array; tiles of 2048
// moved 1.7x the bytes they wrote): the six passes of 32 views of 1920x1080
// over 30M leaves (32M splats, 90M pairs) take 1.53 + 0.50 ms (scatter +
// hist) against 2.04 + 0.81 with 2048-key tiles and a histogram by ballots.
// Up to a few million elements the launches bound it: three per pass (five
// with a device-wide scan of the histogram), and the plan is made by
// segment, not by block (4.7 us; 35-70 us when one thread wrote the entries
// of all of its segment's blocks).  One 1920x1080 view of 1M leaves: 828 ->
// 593 us with the one- and two-launch scans (64 -> 38 launches).
#include <algorithm>

#include "hgs_internal.h"

namespace hgs {

namespace {

constexpr int kT = 512;  // threads of the hist and scatter kernels
constexpr int kWaves = kT / 64;
constexpr int kTile = (int)kSortTile;
constexpr int kItems = kTile / kT;
constexpr int kRadix = 256;
constexpr int kTSmall = 1024;          // threads of the one-workgroup sort
constexpr uint32_t kSortSmall = 8192;  // and its largest segment: 80 KB of LDS, eight pairs a lane
constexpr int kCopies = 16;  // histogram copies: one digit is at most 4-way contended within a wave

__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// The work of one block of a sort: its element range, and its place in the
// histogram (digit d of the block at hist[hbase + d * hstride]).
struct BlockWork {
    uint32_t b0, b1, hbase, hstride, kbase;
    int seg;
};

// False: no work for this block.
__device__ __forceinline__ bool block_work(const SortPlan &p, int nseg, BlockWork &w)
{
    const uint32_t b = blockIdx.x;
    if (b >= p.first[nseg]) return false;
    int lo = 0, hi = nseg - 1;  // the last segment with first <= b (never an empty one)
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.first[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    const SortSeg s = p.seg[lo];
    const uint32_t f = p.first[lo], j = b - f;
    w.seg = lo;
    w.b0 = s.lo + j * s.chunk;
    w.b1 = min(s.hi, w.b0 + s.chunk);
    w.hbase = kRadix * f + j;
    w.hstride = s.nb;
    w.kbase = s.kbase;
    return true;
}

__global__ __launch_bounds__(kT) void k_rs_hist(const uint32_t *__restrict__ keys, int shift, SortPlan plan, int nseg,
                                                uint32_t *__restrict__ hist, uint32_t *__restrict__ tot)
{
    __shared__ uint32_t s_h[kRadix * kCopies];
    BlockWork bw;
    if (!block_work(plan, nseg, bw)) return;
    for (int k = threadIdx.x; k < kRadix * kCopies; k += kT) s_h[k] = 0;
    __syncthreads();
    const uint32_t copy = threadIdx.x & (kCopies - 1);
    for (uint32_t base = bw.b0; base < bw.b1; base += kTile) {
        uint32_t d[kItems];
#pragma unroll
        for (int it = 0; it < kItems; ++it) {  // all loads of the tile in flight at once
            const uint32_t i = base + (uint32_t)(it * kT) + threadIdx.x;
            d[it] = i < bw.b1 ? ((keys[i] - bw.kbase) >> shift) & 0xFFu : 0x100u;
        }
#pragma unroll
        for (int it = 0; it < kItems; ++it)
            if (d[it] < 0x100u) atomicAdd(&s_h[d[it] * kCopies + copy], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kRadix) {
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < kCopies; ++k)
            c += s_h[threadIdx.x * kCopies + ((k + threadIdx.x) & (kCopies - 1))];  // rotated: no bank conflicts
        hist[bw.hbase + threadIdx.x * bw.hstride] = c;
        if (c) atomicAdd(&tot[bw.seg * kRadix + (int)threadIdx.x], c);
    }
}

// One wave per row (segment, digit) of the histogram, in place.
__global__ __launch_bounds__(256) void k_rs_rowscan(SortPlan plan, const uint32_t *__restrict__ tot,
                                                    uint32_t *__restrict__ hist)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int seg = row >> 8, d = row & 255;
    const SortSeg s = plan.seg[seg];
    if (s.nb == 0) return;
    uint32_t base = 0;  // elements of the segment with a lower digit
    {
        const uint4 t = reinterpret_cast<const uint4 *>(tot + seg * kRadix)[lane];
        const int e = 4 * lane;
        base = (e < d ? t.x : 0u) + (e + 1 < d ? t.y : 0u) + (e + 2 < d ? t.z : 0u) + (e + 3 < d ? t.w : 0u);
#pragma unroll
        for (int k = 32; k >= 1; k >>= 1) base += __shfl_xor(base, k, 64);
    }
    uint32_t run = s.lo + base;
    uint32_t *h = hist + (size_t)kRadix * plan.first[seg] + (size_t)d * s.nb;
    for (uint32_t j0 = 0; j0 < s.nb; j0 += 256) {
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t j = j0 + 4u * lane + k;
            v[k] = j < s.nb ? h[j] : 0u;
            sum += v[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const uint32_t y = __shfl_up(inc, k, 64);
            if (lane >= k) inc += y;
        }
        uint32_t ex = run + inc - sum;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t j = j0 + 4u * lane + k;
            if (j < s.nb) h[j] = ex;
            ex += v[k];
        }
        run += __shfl(inc, 63, 64);
    }
}

__global__ __launch_bounds__(kT) void k_rs_scatter(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                   uint32_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                   int shift, SortPlan plan, int nseg,
                                                   const uint32_t *__restrict__ offsets)
{
    __shared__ uint32_t s_keys[kTile];
    __shared__ uint32_t s_vals[kTile];
    __shared__ uint32_t s_wcnt[kWaves][kRadix];
    __shared__ uint32_t s_start[kRadix];  // first tile slot of the digit
    __shared__ uint32_t s_out[kRadix];    // output slot of tile slot 0 if it were the digit's
    __shared__ uint32_t s_w[kRadix / 64];

    BlockWork bw;
    if (!block_work(plan, nseg, bw)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    // thread d < 256 carries the next output slot of digit d
    uint32_t run = threadIdx.x < kRadix ? offsets[bw.hbase + threadIdx.x * bw.hstride] : 0u;

    for (uint32_t base = bw.b0; base < bw.b1; base += kTile) {
#pragma unroll
        for (int k = 0; k < kRadix * kWaves / kT; ++k) (&s_wcnt[0][0])[k * kT + threadIdx.x] = 0;
        uint32_t key[kItems], val[kItems], rank[kItems];
#pragma unroll
        for (int it = 0; it < kItems; ++it) {  // all loads of the tile in flight at once
            const uint32_t i = base + (uint32_t)(w * 64 * kItems + it * 64 + lane);
            const bool valid = i < bw.b1;
            key[it] = valid ? kin[i] : 0u;
            val[it] = valid ? vin[i] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const bool valid = base + (uint32_t)(w * 64 * kItems + it * 64 + lane) < bw.b1;
            const uint32_t d = ((key[it] - bw.kbase) >> shift) & 0xFFu;
            const uint64_t peers = match_digit(d, valid);
            const uint32_t before = s_wcnt[w][d];
            rank[it] = before + (uint32_t)__popcll(peers & lt);
            if (valid && (peers & lt) == 0) s_wcnt[w][d] = before + (uint32_t)__popcll(peers);
            if (!valid) rank[it] = 0xFFFFFFFFu;
        }
        __syncthreads();
        // per digit: wave offsets and tile total, then the exclusive scan of
        // the totals over the digits (one digit per thread)
        uint32_t tot = 0, inc = 0;
        if (threadIdx.x < kRadix) {
            const int d = threadIdx.x;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) {
                const uint32_t c = s_wcnt[k][d];
                s_wcnt[k][d] = tot;
                tot += c;
            }
            inc = tot;
#pragma unroll
            for (int dd = 1; dd < 64; dd <<= 1) {
                const uint32_t y = __shfl_up(inc, dd, 64);
                if (lane >= dd) inc += y;
            }
            if (lane == 63) s_w[w] = inc;
        }
        __syncthreads();
        if (threadIdx.x < kRadix) {
            uint32_t start = inc - tot;
#pragma unroll
            for (int k = 0; k < kRadix / 64; ++k) start += k < w ? s_w[k] : 0u;
            s_start[threadIdx.x] = start;
            s_out[threadIdx.x] = run - start;
            run += tot;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            if (rank[it] == 0xFFFFFFFFu) continue;
            const uint32_t d = ((key[it] - bw.kbase) >> shift) & 0xFFu;
            const uint32_t lp = s_start[d] + s_wcnt[w][d] + rank[it];
            s_keys[lp] = key[it];
            s_vals[lp] = val[it];
        }
        __syncthreads();
        const uint32_t cnt = min((uint32_t)kTile, bw.b1 - base);
#pragma unroll
        for (int it = 0; it < kItems; ++it) {
            const uint32_t j = (uint32_t)(it * kT) + threadIdx.x;
            if (j < cnt) {
                const uint32_t k2 = s_keys[j];
                const uint32_t g = s_out[((k2 - bw.kbase) >> shift) & 0xFFu] + j;
                kout[g] = k2;
                vout[g] = s_vals[j];
            }
        }
        __syncthreads();  // the tile's LDS read before the next tile overwrites it
    }
}

// All passes of a segment of an array of at most kSortSmall places in one
// workgroup: the pairs stay in registers and change places through the LDS,
// ranked as above by (wave, item, lane).  In place.  Bound by the LDS latency of
// one compute unit: 19 us for four passes over 3 k pairs, whose twelve launches
// took 58.
__global__ __launch_bounds__(kTSmall) void k_rs_small(uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                      int passes, SortPlan plan)
{
    constexpr int NW = kTSmall / 64, NI = (int)kSortSmall / kTSmall;
    __shared__ uint32_t s_keys[kSortSmall];
    __shared__ uint32_t s_vals[kSortSmall];
    __shared__ uint32_t s_wcnt[NW][kRadix];
    __shared__ uint32_t s_start[kRadix];
    __shared__ uint32_t s_w[kRadix / 64];

    const SortSeg sg = plan.seg[blockIdx.x];
    if (sg.hi <= sg.lo) return;
    const uint32_t n = min(sg.hi - sg.lo, kSortSmall);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    const int per = (int)((n + kTSmall - 1) / kTSmall);  // items of a lane: the waves share the elements evenly
    const uint32_t i0 = (uint32_t)(w * per * 64 + lane);
    uint32_t key[NI], val[NI], rank[NI];
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const uint32_t i = i0 + it * 64;
        const bool valid = it < per && i < n;
        key[it] = valid ? keys[sg.lo + i] - sg.kbase : 0u;
        val[it] = valid ? vals[sg.lo + i] : 0u;
    }
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
#pragma unroll
        for (int q = 0; q < kRadix * NW / kTSmall; ++q) (&s_wcnt[0][0])[q * kTSmall + threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            if (it >= per) break;
            const bool valid = i0 + it * 64 < n;
            const uint32_t d = (key[it] >> shift) & 0xFFu;
            const uint64_t peers = match_digit(d, valid);
            const uint32_t before = s_wcnt[w][d];
            rank[it] = before + (uint32_t)__popcll(peers & lt);
            if (valid && (peers & lt) == 0) s_wcnt[w][d] = before + (uint32_t)__popcll(peers);
        }
        __syncthreads();
        uint32_t tot = 0, inc = 0;
        if (threadIdx.x < kRadix) {
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                const uint32_t c = s_wcnt[q][threadIdx.x];
                s_wcnt[q][threadIdx.x] = tot;
                tot += c;
            }
            inc = tot;
#pragma unroll
            for (int dd = 1; dd < 64; dd <<= 1) {
                const uint32_t y = __shfl_up(inc, dd, 64);
                if (lane >= dd) inc += y;
            }
            if (lane == 63) s_w[w] = inc;
        }
        __syncthreads();
        if (threadIdx.x < kRadix) {
            uint32_t start = inc - tot;
#pragma unroll
            for (int q = 0; q < kRadix / 64; ++q) start += q < w ? s_w[q] : 0u;
            s_start[threadIdx.x] = start;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            if (it >= per || i0 + it * 64 >= n) break;
            const uint32_t d = (key[it] >> shift) & 0xFFu;
            const uint32_t at = s_start[d] + s_wcnt[w][d] + rank[it];
            s_keys[at] = key[it];
            s_vals[at] = val[it];
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const uint32_t i = i0 + it * 64;
            if (it >= per || i >= n) break;
            key[it] = s_keys[i];
            val[it] = s_vals[i];
        }
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const uint32_t i = i0 + it * 64;
        if (it >= per || i >= n) break;
        keys[sg.lo + i] = key[it] + sg.kbase;
        vals[sg.lo + i] = val[it];
    }
}

// One segment of the whole array.
__global__ __launch_bounds__(kMaxViews) void k_plan_whole(uint32_t cap, const uint32_t *__restrict__ n_dev,
                                                          SortPlan plan, int G, uint32_t *__restrict__ tot,
                                                          uint32_t ntot)
{
    sort_plan_block(0u, min(*n_dev, cap), 0u, min(*n_dev, cap), 1, G, plan, tot, ntot);
}

}  // namespace

int sort_grid(uint32_t cap, int nseg)
{
    // one block per tile up to kSortBlocksMax, and one more per segment (a
    // segment's last chunk is partial)
    const uint64_t want = ((uint64_t)cap + kTile - 1) / kTile + (uint64_t)nseg + 1;
    return (int)std::min<uint64_t>(kSortBlocksMax, want);
}

uint32_t sort_totals(int bits, int nseg) { return (uint32_t)((bits + 7) / 8) * (uint32_t)nseg * kRadix; }

void launch_plan_whole(uint32_t cap, const uint32_t *n_dev, int bits, const SortScratch &s, hipStream_t st)
{
    hipLaunchKernelGGL(k_plan_whole, dim3(1), dim3(kMaxViews), 0, st, cap, n_dev, s.plan, sort_grid(cap, 1), s.tot,
                       sort_totals(bits, 1));
}

// Sorts (keys, vals) over bits [0, bits) with ceil(bits / 8) passes that
// ping-pong between (keys, vals) and the scratch pair, or, if cap is small, in
// place.  Returns true when the sorted result is in (s.k2, s.v2).
bool launch_radix_sort(uint32_t *keys, uint32_t *vals, uint32_t cap, int nseg, int bits, const SortScratch &s,
                       hipStream_t st)
{
    if (cap == 0 || bits <= 0) return false;
    const int passes = (bits + 7) / 8;
    // By the array's capacity, which the host knows, not by the number of pairs,
    // which it does not: no segment can be larger.  So it serves the depth sort
    // while the ctx has rendered nothing larger (its buffers do not shrink) and
    // the sorts of a build; the pair list always has room for more.  One launch
    // instead of three a pass: a render of 4096 leaves (3 k visible) 177 -> 148 us, of 8192
    // visible splats 182 us against 208 with 8193 places and the passes over
    // many blocks, as four views of 2048 against 2049 (184, 221).  Twice as
    // many would fill the LDS and serve one compute unit with twice the work,
    // which is about what the launches cost.
    if (cap <= kSortSmall) {
        hipLaunchKernelGGL(k_rs_small, dim3(nseg), dim3(kTSmall), 0, st, keys, vals, passes, s.plan);
        return false;
    }
    const int G = sort_grid(cap, nseg);
    uint32_t *ki = keys, *vi = vals, *ko = s.k2, *vo = s.v2;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * 8;
        uint32_t *tot = s.tot + (size_t)p * nseg * kRadix;
        hipLaunchKernelGGL(k_rs_hist, dim3(G), dim3(kT), 0, st, ki, shift, s.plan, nseg, s.hist, tot);
        hipLaunchKernelGGL(k_rs_rowscan, dim3(nseg * (kRadix / 4)), dim3(256), 0, st, s.plan, tot, s.hist);
        hipLaunchKernelGGL(k_rs_scatter, dim3(G), dim3(kT), 0, st, ki, vi, ko, vo, shift, s.plan, nseg, s.hist);
        std::swap(ki, ko);
        std::swap(vi, vo);
    }
    return (passes & 1) != 0;
}

}  // namespace hgs
