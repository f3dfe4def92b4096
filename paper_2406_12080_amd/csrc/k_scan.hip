// Device-wide exclusive scan of uint32 counts with a fixed grid, so that the
// element count may live in device memory and the launch sequence can be
// captured in a graph.  Up to kScanSmall elements one block does it; above,
// every block sums its chunk, and a second launch scans it from the sum of
// the chunks before (each block adds those few partial sums itself).
#include "hgs_internal.h"

namespace hgs {

namespace {

constexpr int kT = 256;
constexpr int kItems = 4;
constexpr int kTSmall = 1024;

__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x)
{
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive scan across a block of T threads; *total receives the sum.
template <int T>
__device__ __forceinline__ uint32_t block_exclusive(uint32_t x, uint32_t &total, uint32_t *s_w)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive(x);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < T / 64; ++k) {
        const uint32_t c = s_w[k];
        base += k < w ? c : 0u;
        tot += c;
    }
    __syncthreads();
    total = tot;
    return base + inc - x;
}

__device__ __forceinline__ uint32_t count_of(uint32_t n_host, const uint32_t *n_dev)
{
    return n_dev ? min(*n_dev, n_host) : n_host;
}

// What the scan of the pair counts also notes: the element that holds the
// first pair of every block of `per` pairs below min(total, cap).
struct PairBlocks {
    uint32_t per, cap;
    uint32_t *first;
};

__device__ __forceinline__ void note_blocks(const PairBlocks &pb, uint32_t i, uint32_t o, uint32_t count)
{
    const uint32_t e = min(o + count, pb.cap);
    for (uint32_t b = (o + pb.per - 1) / pb.per; b * pb.per < e; ++b) pb.first[b] = i;
}

// May run in place (in == out): each thread reads its elements before it
// writes them, and no other thread touches them.
__global__ __launch_bounds__(kTSmall) void k_scan_small(const uint32_t *in, uint32_t n_host,
                                                        const uint32_t *__restrict__ n_dev, uint32_t *out,
                                                        uint32_t *__restrict__ total)
{
    __shared__ uint32_t s_w[kTSmall / 64];
    const uint32_t n = count_of(n_host, n_dev);
    uint32_t run = 0;
    for (uint32_t base = 0; base < n; base += kTSmall * kItems) {
        uint32_t v[kItems], s = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint32_t i = base + threadIdx.x * kItems + k;
            v[k] = i < n ? in[i] : 0u;
            s += v[k];
        }
        uint32_t tot;
        uint32_t ex = block_exclusive<kTSmall>(s, tot, s_w) + run;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint32_t i = base + threadIdx.x * kItems + k;
            if (i < n) out[i] = ex;
            ex += v[k];
        }
        run += tot;
    }
    if (threadIdx.x == 0 && total) *total = run;
}

__global__ __launch_bounds__(kT) void k_scan_reduce(const uint32_t *__restrict__ in, uint32_t n_host,
                                                    const uint32_t *__restrict__ n_dev,
                                                    uint32_t *__restrict__ partial)
{
    __shared__ uint32_t s_w[kT / 64];
    const uint32_t n = count_of(n_host, n_dev);
    const uint32_t chunk = (n + kScanBlocks - 1) / kScanBlocks;
    const uint32_t b0 = min(n, blockIdx.x * chunk), b1 = min(n, b0 + chunk);
    uint32_t s = 0;
    for (uint32_t i = b0 + threadIdx.x; i < b1; i += kT) s += in[i];
    uint32_t tot;
    block_exclusive<kT>(s, tot, s_w);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// In place or not, as k_scan_small.
template <bool PAIRS>
__global__ __launch_bounds__(kT) void k_scan_down(const uint32_t *in, uint32_t n_host,
                                                  const uint32_t *__restrict__ n_dev,
                                                  const uint32_t *__restrict__ partial, uint32_t *out,
                                                  uint32_t *__restrict__ total, PairBlocks pb)
{
    __shared__ uint32_t s_w[kT / 64];
    const uint32_t n = count_of(n_host, n_dev);
    const uint32_t chunk = (n + kScanBlocks - 1) / kScanBlocks;
    const uint32_t b0 = min(n, blockIdx.x * chunk), b1 = min(n, b0 + chunk);
    uint32_t before = 0, all = 0;  // the chunks before this one; every chunk
#pragma unroll
    for (int k = 0; k < kScanBlocks / kT; ++k) {
        const uint32_t b = k * kT + threadIdx.x, c = partial[b];
        before += b < blockIdx.x ? c : 0u;
        all += c;
    }
    uint32_t run, tot;
    block_exclusive<kT>(before, run, s_w);
    block_exclusive<kT>(all, tot, s_w);
    if (blockIdx.x == 0 && threadIdx.x == 0 && total) *total = tot;
    for (uint32_t base = b0; base < b1; base += kT * kItems) {
        uint32_t v[kItems];
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint32_t i = base + threadIdx.x * kItems + k;
            v[k] = i < b1 ? in[i] : 0u;
            s += v[k];
        }
        uint32_t tile;
        uint32_t ex = block_exclusive<kT>(s, tile, s_w) + run;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint32_t i = base + threadIdx.x * kItems + k;
            if (i < b1) {
                out[i] = ex;
                if constexpr (PAIRS) note_blocks(pb, i, ex, v[k]);
            }
            ex += v[k];
        }
        run += tile;
    }
}

}  // namespace

void launch_scan(const uint32_t *in, uint32_t n_host, const uint32_t *n_dev, uint32_t *out, uint32_t *total,
                 uint32_t *partial, hipStream_t st)
{
    if (n_host <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(kTSmall), 0, st, in, n_host, n_dev, out, total);
        return;
    }
    hipLaunchKernelGGL(k_scan_reduce, dim3(kScanBlocks), dim3(kT), 0, st, in, n_host, n_dev, partial);
    hipLaunchKernelGGL((k_scan_down<false>), dim3(kScanBlocks), dim3(kT), 0, st, in, n_host, n_dev, partial, out,
                       total, PairBlocks{});
}

void launch_scan_pairs(uint32_t *counts, uint32_t n_host, const uint32_t *n_dev, uint32_t *total, uint32_t *partial,
                       uint32_t pairs_per_block, uint32_t pair_cap, uint32_t *block_first, hipStream_t st)
{
    hipLaunchKernelGGL(k_scan_reduce, dim3(kScanBlocks), dim3(kT), 0, st, counts, n_host, n_dev, partial);
    hipLaunchKernelGGL((k_scan_down<true>), dim3(kScanBlocks), dim3(kT), 0, st, counts, n_host, n_dev, partial,
                       counts, total, PairBlocks{pairs_per_block, pair_cap, block_first});
}

}  // namespace hgs
