// Internal declarations shared by the HIP translation units of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace hgs {

// Conventions of the splatting stage (3D Gaussian splatting defaults that the
// paper's renderer builds on; the 0.99 clamp is the one of Sec. 7.3).
constexpr float kAlphaMin = 1.0f / 255.0f;  // a splat with alpha below this is skipped
constexpr float kTMin = 1e-4f;              // stop before transmittance would fall below
constexpr float kAlphaMax = 0.99f;          // alpha clamp
constexpr double kDilation = 0.3;           // EWA screen-space low-pass variance (px^2)
constexpr int kMaxViews = 1024;

constexpr uint32_t kRootParent = 0x7FFFFFFFu;
constexpr uint32_t kLeafBit = 0x80000000u;

struct DevView {
    float R[9];
    float eye[3];
    float fx, fy, cx, cy;
    int32_t W, H;
    float z_near, tau;
    float cut_klo, cut_khi;  // tau^2 (1 -+ kCutMargin) / max(fx, fy)^2: the cut's FP32 prefilter (NaN: off)
    int32_t tiles_x, tiles_y;
    uint32_t tile_base;  // first global tile id of this view
    uint32_t pix_base;   // first pixel of this view in per-pixel state arrays
    float *out_rgb;      // [H][W][3]
    const float *dL;     // [H][W][3], backward (read) and loss (written) only
    const float *target; // [H][W][3], loss only
};

// Relative band around the cut threshold inside which the FP32 prefilter
// defers to the FP64 evaluation.
constexpr float kCutMargin = 1e-5f;

struct DevHier {
    int64_t n;
    const uint32_t *pinfo;  // parent index | leaf bit
    const float *box;       // [6][n]: bmin x y z, bmax x y z
    const float4 *word_bounds;  // [ceil(n / 64)][2]: bounds of each mask word's parents (k_word_bounds)
    const int32_t *child_count;
    const int32_t *child_begin;  // first child (children are contiguous); 0 for leaves
    const float *mean, *scale, *rot, *opacity, *sh;  // node-major: [N][3] [N][3] [N][4] [N] [N][48]
    // out-of-core rendering: the parameters above are a cache indexed by
    // slot[node] (< 0: not resident); nullptr: indexed by node id
    const int32_t *slot;
};

// Index of a node's parameters (its cache slot when rendering out of core).
__device__ __forceinline__ size_t param_index(const DevHier &h, uint32_t node)
{
    return h.slot ? (size_t)h.slot[node] : (size_t)node;
}

// ---------------------------------------------------- out-of-core rendering
struct StreamParams {
    float *mean, *scale, *rot, *opacity, *sh;  // node-major records (host: N nodes, cache: cap slots)
};
struct StreamDev {
    int32_t *slot;          // [N] cache slot of every node (-1 absent, -2 claimed)
    int32_t *node_in_slot;  // [cap] (-1 free)
    uint32_t *last_used;    // [cap] frame of the last cut that used the slot
    uint32_t *free_stack;   // [cap], free_top entries valid
    uint32_t *free_top, *frame, *req_count, *overflow;
    unsigned long long *transferred;  // total nodes transferred
    uint32_t *req;          // [req_cap] nodes requested this frame
    uint32_t cap, req_cap;
};
void launch_stream_init(const StreamDev &s, int64_t n_nodes, hipStream_t st);
void launch_stream_frame(const StreamDev &s, const uint32_t *pinfo, const int32_t *cut_ids,
                         const uint32_t *cut_total, uint32_t cap, const StreamParams &host,
                         const StreamParams &cache, hipStream_t st);
void launch_stream_cleanup(const StreamDev &s, uint32_t max_age, hipStream_t st);

// Between what lanes of a wave write to the LDS and what others of the same
// wave read there.  The LDS serves a wave in order, so this costs nothing; it
// keeps the compiler from moving either across.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// 32 bits that also hold two 16-bit values written as such.
typedef uint32_t __attribute__((may_alias)) two_u16;

// Blend record of one splat (48 bytes).  The mean is kept as an integer pixel
// anchor plus an FP32 fraction.  The conic (inverse dilated 2D covariance)
// is used through its eigen-axes scaled so that, for a pixel offset d from
// the mean, u_i = w_i . d and G = exp2(-(u_1^2 + u_2^2)) = exp(-d^T conic d / 2):
// a sum of squares, which FP32 evaluates without the cancellation the
// expanded quadratic form suffers for thin splats far from their centre.
struct __align__(16) SplatRec {
    int32_t ax, ay;
    float fx, fy;          // mean - anchor
    float An, Ap;          // kappa |o_n|, kappa |o_p|
    float t, invK;
    float r, g, b;         // -0: infinite (k_blend_end)
    float unused;
};
// The axes w = (w1x, w1y, w2x, w2y) are kept beside the record in FP64
// (double4): the per-8x8-block offsets w . (corner - mean) are formed from
// them in FP64, since a splat's centre can lie far off screen, where the FP32
// rounding of the axis direction alone would move the evaluated position by
// whole 1e-4s; the lanes use their FP32 rounding.
// 1/2 log2(e): exp(-q/2) = exp2(-kHalfLog2e q)
constexpr double kHalfLog2e = 0.72134752044448170368;
static_assert(sizeof(SplatRec) == 48, "record layout");

// Device-side counters of one render.
struct Counters {
    uint32_t cut_total;
    uint32_t vis_total;
    uint32_t pair_total;
    uint32_t overflow;
    uint32_t inf_colour;  // not 0: a visible splat has an infinite colour
    uint32_t pad;
    unsigned long long evaluated;
    unsigned long long blended;
    unsigned long long evaluated_t;      // evaluated pairs of interpolated splats (t > 0)
    unsigned long long bwd_evaluated;    // backward: pairs re-evaluated
    unsigned long long bwd_evaluated_t;
    unsigned long long bwd_contrib;      // backward: pairs that contributed
};

// ---------------------------------------------------------------- launchers
// All launchers queue work on `st`; sizes that only the device knows are read
// from device memory (`*_dev`) and clamped to the host-side capacity.

// cut: per-node predicate over all views, bitmask + per-block counts
constexpr int kCutThreads = 256;
constexpr int kCutItems = 4;
constexpr int kCutBlock = kCutThreads * kCutItems;  // nodes per block
// masks: one bit per (view, node), words * nv; block_counts: per view and
// block of kCutBlock nodes.
// Hierarchy compaction: per-node maximum of eps over a batch of views
// (first batch: written, else folded in), then the keep flags for the
// granularity ladder tau_min 2^i, i < levels.
void launch_compact_emax(const DevHier &h, const DevView *views, int nv, bool first, double *emax, hipStream_t st);
void launch_compact_keep(const DevHier &h, const double *emax, double tau_min, int levels, uint8_t *keep,
                         hipStream_t st);
void launch_cut_flags(const DevHier &h, const DevView *views, int nv, uint64_t *masks, uint32_t *block_counts,
                      int nblocks, hipStream_t st);
// The bounds of every mask word, two float4 each (once per hierarchy).
void launch_word_bounds(const DevHier &h, float4 *bounds, hipStream_t st);
// Also writes word_off[v][w]: the cut position of the first selected node of
// mask word w of view v (words holding a selected node only), and, when
// cut_base is given, cut_base[v] = the cut position of view v's first
// selected node (cut_base[nv] = *cut_total).  Without cut_base nothing is
// written if *cut_total exceeds cap; with it, what fits is.
void launch_cut_emit(const DevHier &h, const DevView *views, int nv, const uint64_t *masks,
                     const uint32_t *block_offsets, int nblocks, uint32_t *word_off, int32_t *out_ids, float *out_t,
                     double *out_t64, uint32_t cap, uint32_t *cut_base, const uint32_t *cut_total, hipStream_t st);

// exclusive scan of uint32; writes *total.  n: min(n_host, *n_dev when given).
// Up to kScanSmall host-side elements in one launch, else two.
void launch_scan(const uint32_t *in, uint32_t n_host, const uint32_t *n_dev, uint32_t *out, uint32_t *total,
                 uint32_t *partial, hipStream_t st);
// The same over the visible splats' tile counts, in place, also noting in
// block_first[b] the splat that holds pair b * pairs_per_block of the list
// the offsets describe, for every block that starts below
// min(total, pair_cap).
void launch_scan_pairs(uint32_t *counts, uint32_t n_host, const uint32_t *n_dev, uint32_t *total, uint32_t *partial,
                       uint32_t pairs_per_block, uint32_t pair_cap, uint32_t *block_first, hipStream_t st);
constexpr int kScanBlocks = 512;
constexpr uint32_t kScanSmall = 16384;

// stable LSD radix sort of (uint32 key, uint32 value) over bit range [0,
// bits), in one or more segments (nseg <= kMaxViews) that are each sorted on
// their own and stay in place, on the digits of key - kbase of the segment
struct SortSeg {
    uint32_t lo, hi;  // elements [lo, hi)
    uint32_t chunk;   // elements per block
    uint32_t nb;      // blocks (0: the segment is empty)
    uint32_t kbase;   // subtracted from every key before the digits are taken
    uint32_t pad[3];
};
struct SortPlan {
    SortSeg *seg;     // [nseg]
    uint32_t *first;  // [nseg + 1]: first block of each segment; [nseg] the blocks used
};
struct SortScratch {
    uint32_t *k2, *v2;  // ping-pong buffers (capacity elements)
    uint32_t *hist;     // 256 * kSortBlocksMax
    uint32_t *tot;      // per pass and segment the 256 digit totals: sort_totals(32, kMaxViews)
    SortPlan plan;      // kMaxViews segments
};
constexpr int kSortBlocksMax = 4096;
constexpr uint32_t kSortTile = 4096;  // keys a block ranks at a time
int sort_grid(uint32_t cap, int nseg);            // blocks of a sort over at most cap elements
uint32_t sort_totals(int bits, int nseg);         // digit totals a sort's plan clears

// The plan of a sort over G blocks, made by one block of kMaxViews threads:
// thread i < nseg gives its segment [lo, hi) (ascending, clamped by the
// caller) and key base; n = all elements.  Every segment gets
// ceil(size / chunk) blocks, the chunk chosen (a multiple of kSortTile) so
// that all segments' blocks fit in G.  Also clears the ntot digit totals.
__device__ __forceinline__ void sort_plan_block(uint32_t lo, uint32_t hi, uint32_t kbase, uint32_t n, int nseg, int G,
                                                const SortPlan &plan, uint32_t *tot, uint32_t ntot)
{
    __shared__ uint32_t s_w[kMaxViews / 64];
    const int i = threadIdx.x, lane = i & 63, w = i >> 6;
    for (uint32_t k = (uint32_t)i; k < ntot; k += kMaxViews) tot[k] = 0u;
    const uint32_t per = max(1u, (n + (uint32_t)(G - nseg) - 1) / (uint32_t)(G - nseg));
    const uint32_t chunk = (per + kSortTile - 1) / kSortTile * kSortTile;
    const uint32_t size = i < nseg ? hi - lo : 0u;
    const uint32_t nb = (size + chunk - 1) / chunk;
    uint32_t inc = nb;  // exclusive scan of the block counts over the segments
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t first = inc - nb, used = 0;
    for (int k = 0; k < kMaxViews / 64; ++k) {
        first += k < w ? s_w[k] : 0u;
        used += s_w[k];
    }
    if (used > (uint32_t)G) used = 0;  // cannot happen for ascending segments; never work past the grid
    if (i < nseg) {
        SortSeg s;
        s.lo = lo;
        s.hi = hi;
        s.chunk = chunk;
        s.nb = used ? nb : 0u;
        s.kbase = kbase;
        s.pad[0] = s.pad[1] = s.pad[2] = 0u;
        plan.seg[i] = s;
        plan.first[i] = used ? first : 0u;
    }
    if (i == 0) plan.first[nseg] = used;
}

// A plan of one segment [0, min(cap, *n_dev)); the sorts of the render path
// make theirs with launch_plan_depth and launch_plan_pairs.
void launch_plan_whole(uint32_t cap, const uint32_t *n_dev, int bits, const SortScratch &s, hipStream_t st);
// Sorts by the plan in s.  Returns true when the sorted result is in
// (s.k2, s.v2).
bool launch_radix_sort(uint32_t *keys, uint32_t *vals, uint32_t cap, int nseg, int bits, const SortScratch &s,
                       hipStream_t st);

// The order of the chunks of 256 cut entries for several views: order[i] = the
// i-th chunk, all views' chunks of one run of nodes together.  order holds
// (cap + 255) / 256 entries and is complete when *cut_total <= cap.
void launch_chunk_order(const uint32_t *block_offsets, int nblocks, int nv, const uint32_t *cut_total,
                        uint32_t *order, uint32_t cap, hipStream_t st);

// preprocess: interpolation, EWA projection, SH colour, footprint, per cut
// entry (order: as above, or NULL: list order)
void launch_preprocess(const DevHier &h, const DevView *views, int nv, const uint32_t *cut_base,
                       const int32_t *cut_ids, const double *cut_t, const uint32_t *cut_total, uint32_t cap,
                       SplatRec *recs, double4 *axes, uint32_t *depth_key, uint4 *trec,
                       float *cjac, uint64_t *vis_mask, uint64_t *pos_mask, uint32_t *vis_block_counts,
                       const uint32_t *order, int tile_w, int tile_h, uint32_t *inf_colour, hipStream_t st);
// Also writes vis_rank[k] = compaction position of visible cut entry k (the
// row of its screen-space gradient).
void launch_compact_visible(const uint64_t *vis_mask, const uint32_t *vis_block_offsets, const uint32_t *cut_total,
                            uint32_t cap, const uint32_t *depth_key, uint32_t *keys, uint32_t *vals,
                            uint32_t *vis_rank, hipStream_t st);
// Tile records of the visible splats in depth order (one gather through
// the sorted values): counts[i] = tile count and rect[i] = tile rectangle of
// the splat at depth slot i, from trec (per cut entry: rect.x, rect.y,
// tile count, unused; written for visible entries).
void launch_gather_tiles(const uint4 *trec, const uint32_t *sorted_vals, const uint32_t *vis_total, uint32_t vis_cap,
                         uint32_t *counts, uint2 *rect, uint32_t *jrank, hipStream_t st);
// The plan of the depth sort: one segment per view, which starts at the
// view's first visible splat (noted in vis_bounds, nv + 1 entries, the last
// = visible total).
void launch_plan_depth(const uint32_t *cut_base, int nv, const uint64_t *vis_mask, const uint32_t *vis_offsets,
                       const uint32_t *cut_total, uint32_t cap, const uint32_t *vis_total, uint32_t *vis_bounds,
                       const SortScratch &s, hipStream_t st);
// The plan of the tile sort: one segment per view, which starts at its first
// (tile, splat) pair; keys count from the view's first global tile id.
void launch_plan_pairs(const uint32_t *vis_bounds, const DevView *views, int nv, const uint32_t *pair_offsets,
                       const uint32_t *vis_total, uint32_t vis_cap, const uint32_t *pair_total, uint32_t pair_cap,
                       int bits, const SortScratch &s, hipStream_t st);
// rect: tile rectangles in depth order (launch_gather_tiles); block_first:
// the splat holding each emission block's first pair (launch_scan_pairs with
// kDupPairs pairs per block; duplicate_blocks(pair_cap) + 1 entries).
constexpr uint32_t kDupPairs = 2048;
void launch_duplicate(const uint2 *rect, const DevView *views, int nv, const uint32_t *cut_base,
                      const uint32_t *sorted_vals, const uint32_t *pair_offsets, const uint32_t *block_first,
                      const uint32_t *vis_total, uint32_t vis_cap, const uint32_t *pair_total, uint32_t pair_cap,
                      uint32_t *pair_keys, uint32_t *pair_vals, Counters *ctr, hipStream_t st);
uint32_t duplicate_blocks(uint32_t pair_cap);
void launch_ranges(const uint32_t *pair_keys, const uint32_t *pair_total, uint32_t pair_cap, uint2 *ranges,
                   hipStream_t st);
void launch_fill_u32(uint32_t *p, uint32_t value, size_t n, hipStream_t st);
// Clears the counters, the tile-length histogram and the tile ranges.
void launch_init(Counters *ctr, uint32_t *tile_hist, uint2 *ranges, uint32_t n_tiles, hipStream_t st);
// Tiles ordered by descending list length (longest first, in steps of an
// eighth of a power of two; any order within a step) for the blend grid.
// tile_hist: 2 kTileBins cleared counters (bin counts, slots taken).
constexpr int kTileBins = 256;
void launch_tile_order(const uint2 *ranges, uint32_t n_tiles, uint32_t *tile_hist, uint32_t *order, hipStream_t st);

// blend (tile_w x tile_h pixels per workgroup)
bool blend_supported(int tw, int th, int batch);
// Looks up the persistent grids of this configuration (device attributes
// and occupancy), so that no such query runs while a launch is captured.
void blend_prepare(int tw, int th);
// persist: a grid of the chip's resident workgroups takes tile slots from
// the device-side queue (*queue, cleared by the launch sequence first)
// instead of one workgroup per tile.
// The deterministic mode of the blend backward (launch_blend_backward with a
// non-NULL DetArgs): per (tile, splat) pair, the tile's 11 screen-space terms
// go to part[11 p] by plain stores, p = the pair's position in the list
// k_duplicate emitted (pair_offsets[j] + the tile's row-major index in the
// tile rectangle rect[j] of depth-sorted visible splat j = jrank[cut entry]);
// launch_det_sum then writes each splat's screen gradient as the in-order sum
// of its pairs' rows.  No floating-point atomics: results are bit-identical
// from run to run.
struct DetArgs {
    const uint32_t *jrank;
    const uint32_t *pair_offsets;
    const uint2 *rect;
    double *part;
};
void launch_det_sum(const double *part, const uint32_t *pair_offsets, const uint32_t *sorted_vals,
                    const uint32_t *vis_rank, const uint32_t *vis_total, uint32_t vis_cap,
                    const uint32_t *pair_total, uint32_t pair_cap, double *sgrad, hipStream_t st);

// Quarter records of the forward, read by the backward: byte b * qstride + p
// (b < the tile's 8x8 blocks, at most kMaxBlocks; qstride >= the pair count)
// holds, for the splat at position p of the sorted pair list and block b of
// its tile, bit q set when some pixel of quarter q of the block blended it
// or stopped at it (a superset of the blends; the backward's per-pixel test
// of the last contributor drops the rest).
constexpr int kMaxBlocks = 8;
void launch_blend(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *tile_order, const uint2 *ranges,
                  const uint32_t *pair_vals,
                  const SplatRec *recs, const double4 *axes, float *T_final, uint32_t *n_last, uint32_t *n_blend,
                  uint8_t *qbits, uint32_t qstride, uint4 *wstats, Counters *ctr, int tw, int th,
                  bool persist, uint32_t *queue, hipStream_t st);

// ---------------------------------------------------- hierarchy generation
// Node arrays of the tree under construction (breadth-first ids).
struct BuildTree {
    int32_t *start, *size;  // first sorted leaf position and leaf count
    int32_t *parent, *child_begin, *child_count;
};
// Leaf inputs, node-major: pos [n][3], scale [n][3], rot [n][4], opacity [n], sh [n][48].
struct BuildLeaves {
    const float *pos, *scale, *rot, *opacity, *sh;
};
// FP64 working values per node (mean [3], cov [6], op, surf, axes [9],
// scales [3], matched R [9] and q [4]) and the interior nodes' SH [48] by
// interior rank.
struct BuildWork {
    double *mean, *cov, *op, *surf, *axes, *sc;
    double *sh;
    int32_t *irank;
    double *R, *q;
};
// FP32 outputs, node-major (bmin / bmax [N][3]).
struct BuildOut {
    float *mean, *scale, *rot, *opacity, *sh, *bmin, *bmax;
};
void build_axis_maps_upload(hipStream_t st);
void launch_build_bounds(const float *pos, int64_t n, float *part, int nblocks, hipStream_t st);
void launch_build_morton(const float *pos, int64_t n, const double lo[3], double s, uint32_t *key_lo,
                         uint32_t *key_hi, uint32_t *idx, hipStream_t st);
void launch_gather_u32(const uint32_t *src, const uint32_t *idx, int64_t n, uint32_t *dst, hipStream_t st);
void launch_split_level(const uint32_t *lo, const uint32_t *hi, int64_t n, uint8_t *sl, hipStream_t st);
void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st);
void launch_level_starts(const int32_t *node_of, const uint8_t *sl, const BuildTree &t, int64_t n, int next_level,
                         uint32_t *flag, hipStream_t st);
void launch_level_nodes(const int32_t *node_of, const uint32_t *flag, const uint32_t *rank, const BuildTree &t,
                        int64_t n, int32_t base, int32_t *node_of_next, hipStream_t st);
void launch_level_sizes(const BuildTree &t, int32_t base, int32_t count, int64_t n, const uint32_t *sorted_idx,
                        int32_t *leaf_src, hipStream_t st);
void launch_interior_ranks(const int32_t *child_count, int64_t N, uint32_t *flag, hipStream_t st);
void launch_interior_list(const int32_t *child_count, const uint32_t *irank, int64_t N, int32_t *interior,
                          hipStream_t st);
void launch_merge_level(const BuildTree &t, const int32_t *leaf_src, const BuildLeaves &in, const BuildWork &w,
                        int32_t base, int32_t count, hipStream_t st);
void launch_match_level(const BuildTree &t, const BuildWork &w, int32_t base, int32_t count, const BuildOut &o,
                        hipStream_t st);
// the SH records of all N nodes, after every level is merged
void launch_out_sh(const BuildTree &t, const BuildWork &w, int64_t N, const BuildOut &o, const int32_t *leaf_src,
                   const float *in_sh, hipStream_t st);
void launch_box_level(const BuildTree &t, int32_t base, int32_t count, float *bmin, float *bmax, hipStream_t st);
// pinfo (parent | leaf bit) and the component-major boxes [6][N] of a built tree
void launch_build_finish(const BuildTree &t, int64_t N, const float *bmin, const float *bmax, uint32_t *pinfo,
                         float *box, hipStream_t st);
// the inverse, for downloads: parent and node-major boxes from pinfo and [6][N]
void launch_unpack_nodes(const uint32_t *pinfo, const float *box, int64_t N, int32_t *parent, float *bmin,
                         float *bmax, hipStream_t st);

// L1 loss of the rendered images (views[v].out_rgb) against views[v].target
// over n_pix pixels of all views: dL/dC written to views[v].dL, the mean
// absolute difference to *loss (device), summed over at most kL1Blocks
// per-block partials (partial: workspace of that many doubles).
// Floats per cut entry of the attribute-gradient rows between the
// preprocess backward and the gradient gather.
constexpr int kPGradFloats = 20;

constexpr int kL1Blocks = 4096;
void launch_l1(const DevView *views, int nv, uint32_t n_pix, double *partial, double *loss, hipStream_t st);

// backward
void launch_blend_backward(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *tile_order,
                           const uint2 *ranges,
                           const uint32_t *pair_vals, const SplatRec *recs, const double4 *axes, const float *T_final,
                           const uint32_t *n_last, const uint8_t *qbits, uint32_t qstride, const uint32_t *vis_rank,
                           double *sgrad, const DetArgs *det, uint4 *wstats,
                           Counters *ctr, int tw, int th, bool want_dt, bool persist, uint32_t *queue,
                           hipStream_t st);
// optimiser step (Adam) over the interior nodes of one parameter group
// (0 mean, 1 scale, 2 rotation, 3 opacity, 4 SH); bc1 = 1 / (1 - beta1^t),
// bc2 = 1 / (1 - beta2^t)
struct AdamScalars {
    float lr, beta1, beta2, eps, bc1, bc2;
};

// One Adam update of one element (the step of 3D Gaussian Splatting's
// optimiser, bias-corrected): the separate optimiser step and the one fused
// into the gradient gather both call it, so that they agree bit for bit.
// The fused multiply-adds are written out and no other contraction is
// allowed: left to the compiler, the choice of which product to fuse
// differed between the two kernels.
__device__ __forceinline__ void adam_one(float &p, float g, float &m, float &v, const AdamScalars &s)
{
#pragma clang fp contract(off)
    m = fmaf(s.beta1, m, (1.0f - s.beta1) * g);
    v = fmaf(s.beta2, v, ((1.0f - s.beta2) * g) * g);
    p -= s.lr * (m * s.bc1) / (sqrtf(v * s.bc2) + s.eps);
}

// The optimiser step fused into the backward's gradient gather: per group
// the parameters (node-major) and both moments (by interior rank), and the
// group's scalars in device memory (5 records, written before each launch).
struct AdamRows {
    float *p[5], *m[5], *v[5];
    const AdamScalars *sc;
};
void launch_zero_rows(double *rows, int width, const uint32_t *vis_total, uint32_t vis_cap, hipStream_t st);
// pos_mask: three words per 64 cut entries, the colour channels above the
// clamp.  order: the forward's, or NULL.  live: a word per 64 cut entries;
// sel: as many words as masks; word_views: per mask word of
// one view a word for every 64 views (all three written here).
void launch_preprocess_backward(const DevHier &h, const DevView *views, int nv, const uint32_t *cut_base,
                                const int32_t *cut_ids, const double *cut_t, const uint32_t *cut_total, uint32_t cap,
                                const uint64_t *vis_mask, const uint64_t *pos_mask, const float *cjac,
                                const uint32_t *vis_offsets,
                                const uint32_t *order, const double *sgrad, float *pg, uint64_t *live,
                                uint64_t *sel, uint64_t *word_views, const uint64_t *masks, int64_t words, const uint32_t *word_off,
                                const int32_t *interior, int64_t n_interior, float *g_mean, float *g_scale,
                                float *g_rot, float *g_opacity, float *g_sh, float *g_dt, const AdamRows *fused,
                                hipStream_t st);

void launch_adam(int group, const int32_t *interior, int64_t n_interior, float *p, float *g, float *m, float *v,
                 const AdamScalars &s, hipStream_t st);

// ------------------------------------------------------------ wave helpers
// Lane exchange through DPP (no LDS traffic); CTRL is a DPP control word:
// 0x128 rotates each row of 16 lanes by 8 (lane l reads l ^ 8), 0x141
// mirrors each half row (l ^ 7), quad permutations 0x4E (l ^ 2) and 0xB1
// (l ^ 1).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ uint64_t lanemask_lt()
{
    const uint32_t lane = __lane_id();
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

}  // namespace hgs
