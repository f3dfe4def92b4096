// Preprocess (one thread per cut entry): interpolation and EWA projection in
// FP64, footprint and tile rectangle, then SH colour (FP32) of the visible
// splats only; then visibility compaction, tile
// counts, pair emission and per-tile ranges.  Also the preprocess backward.
#include <algorithm>

#include "hgs_internal.h"
#include "project.h"

namespace hgs {

namespace {

constexpr int kT = 256;
constexpr double kAlphaMinD = 1.0 / 255.0;
// per cut entry, gradient w.r.t. the interpolated attributes: mean 0..2,
// scale 3..5, raw quaternion 6..9, node opacity 10, parent opacity 11,
// colour cotangent 12..14, view direction 15..17 (the SH basis follows from
// it in the gather, as the forward evaluated it), t 18, 19 unused
constexpr int kPG = kPGradFloats;
static_assert(kPG == 20, "row layout");

// Stores of what only later kernels read: past the L2's reuse, which the
// parameter records need.
typedef float nt_f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_past(float4 *p, const float4 &v)
{
    __builtin_nontemporal_store((nt_f4{v.x, v.y, v.z, v.w}), reinterpret_cast<nt_f4 *>(p));
}

// Writes the rows of Q quads (16 bytes) that lie one behind the other in
// `rows` for the 64 lanes of a wave to out, rows of the lanes in m only: in
// consecutive quads, so that a cache line leaves the wave once and whole
// instead of in Q parts (with the stores past the L2 the forward preprocess
// went from 3.62 to 3.35 ms at 30 M visible splats of 32 views).
template <int Q>
__device__ __forceinline__ void store_rows(const float4 *rows, float4 *out, uint64_t m, int lane)
{
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const uint32_t e = 64u * i + (uint32_t)lane;
        if ((m >> (e / Q)) & 1ull) store_past(out + e, rows[e]);
    }
}

__device__ __forceinline__ int view_of(const uint32_t *cut_base, int nv, uint32_t k)
{
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (cut_base[mid] <= k) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// view_of for the lanes of a wave whose entries are close together: one
// search with the first active lane's entry (a wave-uniform value, so its
// loads go through the scalar cache), and a search of its own only for a
// lane whose entry lies outside that view
__device__ __forceinline__ int view_of_wave(const uint32_t *cut_base, int nv, uint32_t k)
{
    const uint32_t kf = __builtin_amdgcn_readfirstlane(k);
    const int vf = view_of(cut_base, nv, kf);
    const uint32_t b0 = cut_base[vf], b1 = vf + 1 < nv ? cut_base[vf + 1] : 0xFFFFFFFFu;
    return k >= b0 && k < b1 ? vf : view_of(cut_base, nv, k);
}

// The order in which the chunks of kT cut entries are worked on when there are
// several views.  The list is view-major, but the views' cuts hold mostly the
// same nodes (2.3 to 5 views per selected node at 8 to 32 views), 192 B of SH
// and 48 B of geometry each: chunk after chunk of one view, every view reads
// them from memory again (17 GB at 30 M visible splats).  Here all views'
// chunks that begin in a run of kOrderBlocks cut blocks (4096 nodes) follow
// each other, so that the first one's reads serve the others from the L2: at
// 30 M visible splats of 32 views 17.0 -> 11.9 GB read and 4.49 -> 4.06 ms, at
// 8 views of a 3 M node hierarchy 873 -> 775 us.  Runs of 2048 to 16384 nodes
// are alike within the runs' noise (3%).  A single view's list has nothing to
// share and keeps its order.
// One wave per run: lane v holds the chunks of view v that begin there,
// [ceil(a / kT), ceil(b / kT)) with a and b the run's bounds in the view's
// list, and the chunks before them in the order are, over all views, those
// that begin between the view's start and the run.
constexpr int kOrderBlocks = 4;

__global__ __launch_bounds__(kT) void k_chunk_order(const uint32_t *__restrict__ block_offsets, int nblocks, int nv,
                                                    const uint32_t *__restrict__ cut_total,
                                                    uint32_t *__restrict__ order, uint32_t cap_chunks)
{
    const int lane = threadIdx.x & 63;
    const int b0 = (int)(blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * kOrderBlocks;
    if (b0 >= nblocks) return;
    const int b1 = min(b0 + kOrderBlocks, nblocks);
    const int64_t end = (int64_t)nv * nblocks;
    auto first = [&](int64_t i) -> uint32_t {  // the first chunk that begins at or behind offset i
        const uint32_t o = i < end ? block_offsets[i] : *cut_total;
        return o / kT + (o % kT != 0);
    };
    uint32_t before = 0;
    for (int v = lane; v < nv; v += 64) before += first((int64_t)v * nblocks + b0) - first((int64_t)v * nblocks);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) before += (uint32_t)__shfl_xor((int)before, d, 64);
    for (int v0 = 0; v0 < nv; v0 += 64) {
        const int v = v0 + lane;
        uint32_t c = 0, n = 0;
        if (v < nv) {
            c = first((int64_t)v * nblocks + b0);
            n = first((int64_t)v * nblocks + b1) - c;
        }
        uint32_t inc = n;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = (uint32_t)__shfl_up((int)inc, d, 64);
            if (lane >= d) inc += u;
        }
        const uint32_t pos = before + inc - n;
        for (uint32_t i = 0; i < n; ++i)
            if (pos + i < cap_chunks) order[pos + i] = c + i;
        before += (uint32_t)__shfl((int)inc, 63, 64);
    }
}

// Workgroups go round robin over the 8 XCDs, each with an L2 of its own: an
// XCD takes runs of kXcdRun consecutive places of the order (3.53 ms with 64
// or 128, 3.66 with 256, 3.73 with 1024).
constexpr uint32_t kXcdRun = 64;

__host__ __device__ __forceinline__ uint32_t chunk_grid(uint32_t n)
{
    return (n + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun);
}

// The place in the order of workgroup g's chunk (chunk_grid(n) workgroups).
__device__ __forceinline__ uint32_t chunk_place(uint32_t g)
{
    const uint32_t j = g >> 3;
    return ((j / kXcdRun) * 8 + (g & 7u)) * kXcdRun + j % kXcdRun;
}

template <bool SH_ALIGNED>
__global__ __launch_bounds__(kT, 4) void k_preprocess(DevHier h, const DevView *__restrict__ views, int nv,
                                                   const uint32_t *__restrict__ cut_base,
                                                   const int32_t *__restrict__ cut_ids,
                                                   const double *__restrict__ cut_t,
                                                   const uint32_t *__restrict__ cut_total, uint32_t cap,
                                                   SplatRec *__restrict__ recs, double4 *__restrict__ axes,
                                                   uint32_t *__restrict__ depth_key,
                                                   uint4 *__restrict__ trec,
                                                   float *__restrict__ cjac, uint64_t *__restrict__ vis_mask,
                                                   uint64_t *__restrict__ pos_mask,
                                                   uint32_t *__restrict__ vis_block_counts,
                                                   const uint32_t *__restrict__ order, int tile_w, int tile_h,
                                                   uint32_t *__restrict__ inf_colour)
{
    __shared__ __align__(16) char s_sh[kT / 64][kShStage];
    __shared__ uint2 s_src[kT / 64][64];
    __shared__ uint32_t s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    const uint32_t cut = *cut_total, total = min(cut, cap);
    const uint32_t nchunks = (total + kT - 1) / kT, cap_chunks = (cap + kT - 1) / kT;
    uint32_t chunk = blockIdx.x;
    if (order && cut <= cap) {  // (a cut beyond the capacity is rendered again: any order)
        // chunks behind the cut stay with the workgroup of their number
        if (blockIdx.x >= nchunks && blockIdx.x < cap_chunks) {
            if (threadIdx.x < kT / 64 && blockIdx.x * kT + 64 * threadIdx.x < cap)
                vis_mask[blockIdx.x * (kT / 64) + threadIdx.x] = 0ull;
            if (threadIdx.x == 0) vis_block_counts[blockIdx.x] = 0u;
        }
        const uint32_t at = chunk_place(blockIdx.x);
        if (at >= nchunks) return;
        chunk = order[at];
    }
    if (chunk >= cap_chunks) return;
    const uint32_t k = chunk * kT + threadIdx.x;
    bool vis = false;
    SplatRec r;
    double4 ax4 = make_double4(0.0, 0.0, 0.0, 0.0);
    size_t pn = 0, pp = 0;  // parameter records of the node and, with t > 0, its parent
    float dir[3] = {0.0f, 0.0f, 0.0f}, t = 0.0f;
    if (k < total) {
        const int vi = view_of_wave(cut_base, nv, k);
        const DevView &V = views[vi];
        Proj P;
        project_splat(h, V, (uint32_t)cut_ids[k], cut_t[k], P);
        if (P.ok) {
            // footprint: alpha <= min(0.99, A G) with A = kappa((1-t)o_n + t o_p);
            // alpha_min can only be reached inside d^T Sigma2'^-1 d <= 2 ln(A/alpha_min)
            const double A = P.kappa * ((1.0 - P.t) * P.o_n + P.t * P.o_p);
            if (A >= kAlphaMinD && fabs(P.u) < 1e9 && fabs(P.v) < 1e9) {
                const double r2 = 2.0 * log(A / kAlphaMinD);
                const double hx = sqrt(r2 * (P.a + kDilation)), hy = sqrt(r2 * (P.c + kDilation));
                double x0 = ceil(P.u - hx - 0.5), x1 = floor(P.u + hx - 0.5);
                double y0 = ceil(P.v - hy - 0.5), y1 = floor(P.v + hy - 0.5);
                x0 = fmax(x0, 0.0);
                y0 = fmax(y0, 0.0);
                x1 = fmin(x1, (double)(V.W - 1));
                y1 = fmin(y1, (double)(V.H - 1));
                if (x1 >= x0 && y1 >= y0) {
                    vis = true;
                    const uint32_t tx0 = (uint32_t)x0 / tile_w, tx1 = (uint32_t)x1 / tile_w;
                    const uint32_t ty0 = (uint32_t)y0 / tile_h, ty1 = (uint32_t)y1 / tile_h;
                    const uint32_t nt = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
                    trec[k] = make_uint4(tx0 | (tx1 << 16), ty0 | (ty1 << 16), nt, 0u);
                    const double fu = floor(P.u), fv = floor(P.v);
                    r.ax = (int32_t)fu;
                    r.ay = (int32_t)fv;
                    r.fx = (float)(P.u - fu);
                    r.fy = (float)(P.v - fv);
                    // eigen-axes of the conic [[ca, cb], [cb, cc]]: the major axis at
                    // angle th with (cos 2th, sin 2th) = (ca - cc, 2 cb) / r, its cosine
                    // and sine by the half-angle formulas (each from the better
                    // conditioned one), th in (-pi/2, pi/2]; any direction for a circle
                    const double ca = P.conic[0], cb = P.conic[1], cc = P.conic[2];
                    const double dx = ca - cc, dy = 2.0 * cb, rr = sqrt(dx * dx + dy * dy);
                    double cs = 1.0, sn = 0.0;
                    if (rr > 0.0) {
                        const double c2 = dx / rr, s2 = dy / rr;
                        if (c2 >= 0.0) {
                            cs = sqrt(0.5 * (1.0 + c2));
                            sn = s2 / (2.0 * cs);
                        } else {
                            sn = copysign(sqrt(0.5 * (1.0 - c2)), s2);
                            cs = s2 / (2.0 * sn);
                        }
                    }
                    const double l1 = ca * cs * cs + 2.0 * cb * sn * cs + cc * sn * sn;
                    const double l2 = ca * sn * sn - 2.0 * cb * sn * cs + cc * cs * cs;
                    const double s1 = sqrt(fmax(l1, 0.0) * kHalfLog2e), s2 = sqrt(fmax(l2, 0.0) * kHalfLog2e);
                    ax4 = make_double4(s1 * cs, s1 * sn, -s2 * sn, s2 * cs);
                    r.An = (float)(P.kappa * P.o_n);
                    r.Ap = (float)(P.kappa * P.o_p);
                    r.t = (float)P.t;
                    r.invK = (float)(1.0 / (double)P.K);
                    depth_key[k] = __float_as_uint((float)P.pc[2]);
                    pn = P.pn;
                    pp = P.use_par ? P.pp : P.pn;
                    t = (float)P.t;
#pragma unroll
                    for (int c = 0; c < 3; ++c) dir[c] = (float)P.dir[c];
                }
            }
        }
    }
    const uint64_t m = __ballot(vis);
    if (m) {
        float raw[3] = {0.0f, 0.0f, 0.0f}, dcol[3][3], dpn[3];
        const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
        splat_colour<SH_ALIGNED>(h.sh, vis, pn, pp, t, dir, s_sh[w], s_src[w], raw, dcol, dpn);
        // the channels above the colour's clamp at zero
        const uint64_t p0 = __ballot(vis && raw[0] > 0.0f), p1 = __ballot(vis && raw[1] > 0.0f),
                       p2 = __ballot(vis && raw[2] > 0.0f);
        if (lane < 3) pos_mask[(size_t)(k >> 6) * 3 + lane] = lane == 0 ? p0 : (lane == 1 ? p1 : p2);
        if (vis) {
            auto clamp = [&](float c) -> float {  // at 0 (NaN too); an infinite colour as -0, and noted
                if (c == __builtin_inff()) {
                    *inf_colour = 1u;
                    return -0.0f;
                }
                return fabsf(fmaxf(c, 0.0f));
            };
            r.r = clamp(raw[0]);
            r.g = clamp(raw[1]);
            r.b = clamp(raw[2]);
            r.unused = 0.0f;
        }
        // record, colour Jacobian and axes, row by row through the LDS
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wave_lds_sync();
        float4 *o = reinterpret_cast<float4 *>(s_sh[w]);
        static_assert(sizeof(SplatRec) == 48 && kShStage >= 64 * (48 + 48 + 32), "rows of 3, 3 and 2 quads");
        if (vis) {
            __builtin_memcpy(o + 3 * lane, &r, sizeof r);
            o[192 + 3 * lane] = make_float4(dcol[0][0], dcol[0][1], dcol[0][2], dcol[1][0]);
            o[193 + 3 * lane] = make_float4(dcol[1][1], dcol[1][2], dcol[2][0], dcol[2][1]);
            o[194 + 3 * lane] = make_float4(dcol[2][2], dpn[0], dpn[1], dpn[2]);
            __builtin_memcpy(o + 384 + 2 * lane, &ax4, sizeof ax4);
        }
        wave_lds_sync();
        const size_t kw = k & ~63u;
        store_rows<3>(o, reinterpret_cast<float4 *>(recs + kw), m, lane);
        store_rows<3>(o + 192, reinterpret_cast<float4 *>(cjac + 12 * kw), m, lane);
        store_rows<2>(o + 384, reinterpret_cast<float4 *>(axes + kw), m, lane);
    }
    const uint32_t k0 = chunk * kT + (threadIdx.x & ~63u);
    if ((threadIdx.x & 63) == 0) {
        if (k0 < cap) vis_mask[k0 >> 6] = m;
        if (m) atomicAdd(&s_cnt, (uint32_t)__popcll(m));
    }
    __syncthreads();
    if (threadIdx.x == 0) vis_block_counts[chunk] = s_cnt;
}

__global__ __launch_bounds__(kT) void k_compact_visible(const uint64_t *__restrict__ vis_mask,
                                                        const uint32_t *__restrict__ offsets,
                                                        const uint32_t *__restrict__ cut_total, uint32_t cap,
                                                        const uint32_t *__restrict__ depth_key,
                                                        uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                        uint32_t *__restrict__ vis_rank)
{
    const uint32_t total = min(*cut_total, cap);
    const uint32_t k = blockIdx.x * kT + threadIdx.x;
    if (blockIdx.x * kT >= total) return;
    __shared__ uint32_t s_pre[kT / 64];
    __shared__ uint64_t s_m[kT / 64];
    if (threadIdx.x < kT / 64) s_m[threadIdx.x] = vis_mask[blockIdx.x * (kT / 64) + threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int w = 0; w < kT / 64; ++w) {
            s_pre[w] = acc;
            acc += (uint32_t)__popcll(s_m[w]);
        }
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, bit = threadIdx.x & 63;
    const uint64_t m = s_m[w];
    if (k < total && ((m >> bit) & 1ull)) {
        const uint32_t pos = offsets[blockIdx.x] + s_pre[w] + (uint32_t)__popcll(m & ((1ull << bit) - 1ull));
        keys[pos] = depth_key[k];
        vals[pos] = k;
        vis_rank[k] = pos;
    }
}

// The plan of the depth sort: one segment per view.  A view's first visible
// splat sits behind the visible entries before cut position cut_base[v] (the
// visible list keeps the cut's view-major order).
__global__ __launch_bounds__(kMaxViews) void k_plan_depth(const uint32_t *__restrict__ cut_base, int nv,
                                                          const uint64_t *__restrict__ vis_mask,
                                                          const uint32_t *__restrict__ vis_offsets,
                                                          const uint32_t *__restrict__ cut_total, uint32_t cap,
                                                          const uint32_t *__restrict__ vis_total,
                                                          uint32_t *__restrict__ bounds, SortPlan plan, int G,
                                                          uint32_t *__restrict__ tot, uint32_t ntot)
{
    const uint32_t total = min(*cut_total, cap), nvis = min(*vis_total, cap);
    auto bound = [&](int v) -> uint32_t {
        const uint32_t k = v < nv ? cut_base[v] : total;
        if (k >= total) return nvis;
        uint32_t c = vis_offsets[k / kT];  // visible entries of the preprocess blocks before k's
        for (uint32_t w = (k / kT) * (kT / 64); w < (k >> 6); ++w) c += (uint32_t)__popcll(vis_mask[w]);
        if (k & 63u) c += (uint32_t)__popcll(vis_mask[k >> 6] & ((1ull << (k & 63u)) - 1ull));
        return min(c, nvis);
    };
    const int v = threadIdx.x;
    uint32_t lo = 0, hi = 0;
    if (v < nv) {
        lo = bound(v);
        hi = bound(v + 1);
        bounds[v] = lo;
    }
    if (v == 0) bounds[nv] = nvis;
    sort_plan_block(lo, hi, 0u, nvis, nv, G, plan, tot, ntot);
}

// The plan of the tile sort: one segment per view, its keys counted from the
// view's first global tile id.
__global__ __launch_bounds__(kMaxViews) void k_plan_pairs(const uint32_t *__restrict__ vis_bounds,
                                                          const DevView *__restrict__ views, int nv,
                                                          const uint32_t *__restrict__ pair_offsets,
                                                          const uint32_t *__restrict__ vis_total, uint32_t vis_cap,
                                                          const uint32_t *__restrict__ pair_total, uint32_t pair_cap,
                                                          SortPlan plan, int G, uint32_t *__restrict__ tot,
                                                          uint32_t ntot)
{
    const uint32_t nvis = min(*vis_total, vis_cap), npairs = min(*pair_total, pair_cap);
    auto bound = [&](int v) -> uint32_t {
        const uint32_t j = vis_bounds[v];
        return j < nvis ? min(pair_offsets[j], npairs) : npairs;
    };
    const int v = threadIdx.x;
    uint32_t lo = 0, hi = 0, base = 0;
    if (v < nv) {
        lo = bound(v);
        hi = bound(v + 1);
        base = views[v].tile_base;
    }
    sort_plan_block(lo, hi, base, npairs, nv, G, plan, tot, ntot);
}

// The tile records of the visible splats in depth order: the one random
// gather of per-splat data between the depth sort and the pair emission;
// also each cut entry's depth-order slot (jrank), which the deterministic
// backward uses to find a pair's position in the emitted list.
__global__ __launch_bounds__(kT) void k_gather_tiles(const uint4 *__restrict__ trec,
                                                     const uint32_t *__restrict__ sorted_vals,
                                                     const uint32_t *__restrict__ vis_total, uint32_t vis_cap,
                                                     uint32_t *__restrict__ counts, uint2 *__restrict__ rect,
                                                     uint32_t *__restrict__ jrank)
{
    const uint32_t n = min(*vis_total, vis_cap);
    const uint32_t i = blockIdx.x * kT + threadIdx.x;
    if (i >= n) return;
    const uint32_t s = sorted_vals[i];
    const uint4 r = trec[s];
    counts[i] = r.z;
    rect[i] = make_uint2(r.x, r.y);
    jrank[s] = i;
}

// Deterministic mode: the screen gradient of depth-sorted visible splat j is
// the sum, in emission order, of the rows its pairs' tiles stored (every row
// of the emitted list is written by the backward or zeroed before it).
__global__ __launch_bounds__(kT) void k_det_sum(const double *__restrict__ part,
                                                const uint32_t *__restrict__ pair_offsets,
                                                const uint32_t *__restrict__ sorted_vals,
                                                const uint32_t *__restrict__ vis_rank,
                                                const uint32_t *__restrict__ vis_total, uint32_t vis_cap,
                                                const uint32_t *__restrict__ pair_total, uint32_t pair_cap,
                                                double *__restrict__ sgrad)
{
    const uint32_t n = min(*vis_total, vis_cap);
    const uint32_t j = blockIdx.x * kT + threadIdx.x;
    if (j >= n) return;
    const uint32_t p0 = min(pair_offsets[j], pair_cap);
    const uint32_t p1 = min(j + 1 < n ? pair_offsets[j + 1] : *pair_total, pair_cap);
    double acc[11];
#pragma unroll
    for (int k = 0; k < 11; ++k) acc[k] = 0.0;
    for (uint32_t p = p0; p < p1; ++p) {
        const double *row = part + (size_t)p * 11;
#pragma unroll
        for (int k = 0; k < 11; ++k) acc[k] += row[k];
    }
    double *o = sgrad + (size_t)vis_rank[sorted_vals[j]] * 12;
#pragma unroll
    for (int k = 0; k < 11; ++k) o[k] = acc[k];
    o[11] = 0.0;
}

// Pair emission, balanced by pairs: block b writes pairs [b P, (b + 1) P)
// of the depth-ordered list, whatever the footprints of the splats they come
// from (the nearest splats of every view sort first and may cover thousands
// of tiles each).  The scan of the pair counts noted the splat that holds
// each block's first pair; the block's slice of the pair offsets is staged
// in LDS.
// Each thread writes kDupPer consecutive pairs (one vector store per array
// and thread, contiguous across the wave): a binary search finds the splat
// of its first pair, then it walks forward tile by tile.
constexpr int kDupPer = 8;
static_assert(kDupPairs == (uint32_t)kT * kDupPer, "pairs per emission block");

__global__ __launch_bounds__(kT) void k_duplicate(const uint2 *__restrict__ rect, const DevView *__restrict__ views,
                                                  int nv, const uint32_t *__restrict__ cut_base,
                                                  const uint32_t *__restrict__ sorted_vals,
                                                  const uint32_t *__restrict__ offsets,
                                                  const uint32_t *__restrict__ block_first,
                                                  const uint32_t *__restrict__ vis_total, uint32_t vis_cap,
                                                  const uint32_t *__restrict__ pair_total, uint32_t pair_cap,
                                                  uint32_t *__restrict__ pair_keys, uint32_t *__restrict__ pair_vals,
                                                  Counters *__restrict__ ctr)
{
    __shared__ uint32_t s_off[kDupPairs + 1];
    __shared__ uint32_t s_cb[kMaxViews + 1];
    if (blockIdx.x == 0 && threadIdx.x == 0 && *pair_total > pair_cap) atomicOr(&ctr->overflow, 4u);
    const uint32_t nvis = min(*vis_total, vis_cap);
    const uint32_t npairs = min(*pair_total, pair_cap);
    const uint32_t o0 = blockIdx.x * kDupPairs;
    if (o0 >= npairs || nvis == 0) return;
    const uint32_t o1 = min(o0 + kDupPairs, npairs);
    const uint32_t j0 = block_first[blockIdx.x];
    // last splat that can hold one of the block's pairs: the one holding pair
    // o1 (or the last splat); never more than kDupPairs past j0, since every
    // splat has at least one pair (this also bounds the LDS slice when the
    // pair count exceeded the capacity)
    uint32_t j1 = o1 < npairs ? block_first[blockIdx.x + 1] : nvis - 1;
    j1 = min(j1, j0 + kDupPairs);
    const uint32_t cnt = j1 - j0 + 1;
    for (uint32_t k = threadIdx.x; k < cnt; k += kT) s_off[k] = offsets[j0 + k];
    for (int k = threadIdx.x; k <= nv; k += kT) s_cb[k] = cut_base[k];
    __syncthreads();
    const uint32_t ob = o0 + threadIdx.x * kDupPer;
    if (ob >= o1) return;
    uint32_t lo = 0, hi = cnt - 1;  // the last slot with s_off <= ob
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1u) >> 1;
        if (s_off[mid] <= ob) lo = mid;
        else hi = mid - 1u;
    }
    uint32_t key[kDupPer], val[kDupPer];
    uint32_t cur = ~0u, s = 0, tx = 0, ty = 0, tx0 = 0, tx1 = 0, base = 0, tiles_x = 0;
#pragma unroll
    for (int k = 0; k < kDupPer; ++k) {
        const uint32_t o = ob + k;
        if (o < o1) {
            while (lo + 1u < cnt && s_off[lo + 1u] <= o) ++lo;
            if (lo != cur) {  // first pair of this thread from splat slot lo
                cur = lo;
                s = sorted_vals[j0 + lo];
                int vlo = 0, vhi = nv - 1;  // view of cut entry s
                while (vlo < vhi) {
                    const int mid = (vlo + vhi + 1) >> 1;
                    if (s_cb[mid] <= s) vlo = mid;
                    else vhi = mid - 1;
                }
                const DevView &V = views[vlo];
                base = V.tile_base;
                tiles_x = (uint32_t)V.tiles_x;
                const uint2 r = rect[j0 + lo];
                tx0 = r.x & 0xFFFFu;
                tx1 = r.x >> 16;
                const uint32_t w = tx1 - tx0 + 1u, q = o - s_off[lo];
                ty = (r.y & 0xFFFFu) + q / w;
                tx = tx0 + q % w;
            } else if (++tx > tx1) {  // next tile of the same splat, row by row
                tx = tx0;
                ++ty;
            }
        }
        key[k] = base + ty * tiles_x + tx;
        val[k] = s;
    }
    if (ob + kDupPer <= o1) {
        uint4 *kd = reinterpret_cast<uint4 *>(pair_keys + ob), *vd = reinterpret_cast<uint4 *>(pair_vals + ob);
#pragma unroll
        for (int k = 0; k < kDupPer / 4; ++k) {
            kd[k] = make_uint4(key[4 * k], key[4 * k + 1], key[4 * k + 2], key[4 * k + 3]);
            vd[k] = make_uint4(val[4 * k], val[4 * k + 1], val[4 * k + 2], val[4 * k + 3]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kDupPer; ++k)
            if (ob + k < o1) {
                pair_keys[ob + k] = key[k];
                pair_vals[ob + k] = val[k];
            }
    }
}

// Zeroes the first (visible count) x width doubles of `rows` (the screen
// gradients, one row per visible splat by visible rank).
__global__ __launch_bounds__(kT) void k_zero_rows(double *__restrict__ rows, int width,
                                                  const uint32_t *__restrict__ vis_total, uint32_t vis_cap)
{
    const size_t n = (size_t)min(*vis_total, vis_cap) * (size_t)width;
    for (size_t e = (size_t)blockIdx.x * kT + threadIdx.x; e < n; e += (size_t)gridDim.x * kT) rows[e] = 0.0;
}

// Tile ranges of the sorted pair keys: four keys per thread (one vector
// load), boundaries found against the neighbours.  Tile ids stay below
// 2^31, so ~0 marks "no neighbour".
constexpr int kRangeItems = 4;

__global__ __launch_bounds__(kT) void k_ranges(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ total,
                                               uint32_t cap, uint2 *__restrict__ ranges)
{
    const uint32_t n = min(*total, cap);
    const uint32_t i0 = (blockIdx.x * kT + threadIdx.x) * kRangeItems;
    if (i0 >= n) return;
    uint32_t k[kRangeItems + 2];  // keys[i0 - 1 .. i0 + kRangeItems]
    k[0] = i0 > 0 ? keys[i0 - 1] : ~0u;
    if (i0 + kRangeItems <= n) {
        const uint4 v = *reinterpret_cast<const uint4 *>(keys + i0);
        k[1] = v.x;
        k[2] = v.y;
        k[3] = v.z;
        k[4] = v.w;
    } else {
#pragma unroll
        for (int j = 0; j < kRangeItems; ++j) k[1 + j] = i0 + j < n ? keys[i0 + j] : ~0u;
    }
    k[kRangeItems + 1] = i0 + kRangeItems < n ? keys[i0 + kRangeItems] : ~0u;
#pragma unroll
    for (int j = 0; j < kRangeItems; ++j) {
        const uint32_t i = i0 + j, t = k[1 + j];
        if (i >= n) break;
        if (k[j] != t) ranges[t].x = i;
        if (k[2 + j] != t) ranges[t].y = i + 1;
    }
}

// Scheduling order of the tiles, longest lists first: 256 bins of 255 minus
// 8 log2(list length + 1), counted (k_tile_bins) and filled (k_tile_place).
// The order inside a bin is whatever the blocks' reservations give: it only
// decides which tile a workgroup takes when.  Two launches (8 us for a view
// of 8160 tiles; a radix pass over the bins took five).
constexpr int kTilePer = 4;  // tiles per thread
constexpr int kTileBlock = kT * kTilePer;

__device__ __forceinline__ uint32_t tile_bin(const uint2 r)
{
    const uint32_t len = r.y - r.x + 1u;
    const uint32_t lg = 31u - (uint32_t)__clz(len);  // floor(log2)
    const uint32_t frac = lg >= 3 ? (len >> (lg - 3)) & 7u : (len << (3 - lg)) & 7u;
    return 255u - min(255u, lg * 8u + frac);
}

__global__ __launch_bounds__(kT) void k_tile_bins(const uint2 *__restrict__ ranges, uint32_t n_tiles,
                                                  uint32_t *__restrict__ hist)
{
    __shared__ uint32_t s_h[kTileBins];
    s_h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const uint32_t i = blockIdx.x * kTileBlock + k * kT + threadIdx.x;
        if (i < n_tiles) atomicAdd(&s_h[tile_bin(ranges[i])], 1u);
    }
    __syncthreads();
    if (s_h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], s_h[threadIdx.x]);
}

// hist: the bins' counts; next: kTileBins cleared counters of the slots
// taken in each bin.
__global__ __launch_bounds__(kT) void k_tile_place(const uint2 *__restrict__ ranges, uint32_t n_tiles,
                                                   const uint32_t *__restrict__ hist, uint32_t *__restrict__ next,
                                                   uint32_t *__restrict__ order)
{
    static_assert(kTileBins == kT, "one bin per thread");
    __shared__ uint32_t s_h[kTileBins], s_w[kT / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    s_h[t] = 0;
    const uint32_t all = hist[t];
    uint32_t inc = all;  // first slot of bin t: exclusive scan of the counts
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t first = inc - all;
#pragma unroll
    for (int k = 0; k < kT / 64; ++k) first += k < w ? s_w[k] : 0u;
    uint32_t bin[kTilePer], rank[kTilePer];
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const uint32_t i = blockIdx.x * kTileBlock + k * kT + t;
        bin[k] = i < n_tiles ? tile_bin(ranges[i]) : ~0u;
        if (bin[k] != ~0u) rank[k] = atomicAdd(&s_h[bin[k]], 1u);
    }
    __syncthreads();
    const uint32_t c = s_h[t];
    const uint32_t got = c ? atomicAdd(&next[t], c) : 0u;
    __syncthreads();
    s_h[t] = first + got;  // where this block's tiles of the bin go
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTilePer; ++k)
        if (bin[k] != ~0u) order[s_h[bin[k]] + rank[k]] = blockIdx.x * kTileBlock + k * kT + t;
}

// Clears what a render counts into: the counters, the tile-length bins and
// the tile ranges.
__global__ __launch_bounds__(kT) void k_init(uint32_t *__restrict__ ctr, uint32_t nctr, uint32_t *__restrict__ bins,
                                             uint32_t nbins, uint2 *__restrict__ ranges, uint32_t n_tiles)
{
    for (uint32_t i = blockIdx.x * kT + threadIdx.x; i < n_tiles; i += gridDim.x * kT) ranges[i] = make_uint2(0u, 0u);
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < nctr; i += kT) ctr[i] = 0u;
        for (uint32_t i = threadIdx.x; i < nbins; i += kT) bins[i] = 0u;
    }
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, uint32_t value, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// ------------------------------------------------------------------ backward
// The attribute-gradient row of cut entry k of view V and its dL/dt, if it
// projects and its screen-gradient row is not all zeros (`any`), from its screen-gradient row sg, its colour Jacobian
// cj (both in LDS) and the words pos of its colour channels above the clamp.
__device__ __forceinline__ void entry_bwd(const DevHier &h, const DevView &V, uint32_t k, uint32_t node_id,
                                          double t_in, const uint64_t *__restrict__ pos, const double *sg,
                                          const float *cj, float (&row)[kPG], bool &any, float &dt_out)
{
    Proj P;
    project_splat(h, V, node_id, t_in, P);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the LDS rows have arrived
    if (!P.ok) return;
    const double du = sg[0], dv = sg[1], dAn = sg[5], dAp = sg[6];
    const double drgb[3] = {sg[7], sg[8], sg[9]};
    double dt = sg[10];
    any = !(du == 0.0 && dv == 0.0 && sg[2] == 0.0 && sg[3] == 0.0 && sg[4] == 0.0 && dAn == 0.0 && dAp == 0.0 &&
            drgb[0] == 0.0 && drgb[1] == 0.0 && drgb[2] == 0.0 && dt == 0.0);
    if (!any) return;
    const uint32_t node = P.node, par = P.par;
    const bool use_par = P.has_par && P.t > 0.0;
    const double t = P.t, w0 = 1.0 - t;

    // colour: rgb = max(0, raw); the forward kept raw > 0, d raw / d dir and
    // (SH_p - SH_n) . Y per channel
    double gr[3];
    gr[0] = (pos[0] >> (k & 63u)) & 1ull ? drgb[0] : 0.0;
    gr[1] = (pos[1] >> (k & 63u)) & 1ull ? drgb[1] : 0.0;
    gr[2] = (pos[2] >> (k & 63u)) & 1ull ? drgb[2] : 0.0;
    double ddir[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        ddir[0] += gr[c] * (double)cj[3 * c];
        ddir[1] += gr[c] * (double)cj[3 * c + 1];
        ddir[2] += gr[c] * (double)cj[3 * c + 2];
        if (use_par) dt += gr[c] * (double)cj[9 + c];
    }
    row[15] = (float)P.dir[0];
    row[16] = (float)P.dir[1];
    row[17] = (float)P.dir[2];
    row[18] = (float)t;
    row[12] = (float)gr[0];
    row[13] = (float)gr[1];
    row[14] = (float)gr[2];
    double dmu[3];
    {
        const double dd = P.dir[0] * ddir[0] + P.dir[1] * ddir[1] + P.dir[2] * ddir[2];
#pragma unroll
        for (int m = 0; m < 3; ++m) dmu[m] = (ddir[m] - P.dir[m] * dd) / P.rlen;
    }

    // A_n = kappa o_n, A_p = kappa o_p
    const double dkappa = dAn * P.o_n + dAp * P.o_p;
    const double don = dAn * P.kappa, dop = dAp * P.kappa;

    // dL/d(a, b, c) of Sigma2 through the conic arrives accumulated per pixel
    // (the blend backward sums -dL/dq (conic d)(conic d)^T); add the part
    // through kappa = sqrt(det Sigma2 / det(Sigma2 + hI))
    const double a = P.a, b = P.b, c = P.c;
    const double ad = a + kDilation, cd = c + kDilation;
    const double Dd = P.Dd, D = P.D;
    double da = sg[2], db = sg[3], dc = sg[4];
    if (D > 0.0 && P.kappa > 0.0) {
        const double hk = 0.5 * P.kappa * dkappa;
        da += hk * (c / D - cd / Dd);
        dc += hk * (a / D - ad / Dd);
        db += hk * (2.0 * b / Dd - 2.0 * b / D);
    }

    // Sigma2 = Tm Sigma3 Tm^T
    const double *T0 = P.Tm, *T1 = P.Tm + 3;
    const double *S = P.cov3;
    const double Sf[9] = {S[0], S[1], S[2], S[1], S[3], S[4], S[2], S[4], S[5]};
    double T0S[3], T1S[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        T0S[j] = T0[0] * Sf[j] + T0[1] * Sf[3 + j] + T0[2] * Sf[6 + j];
        T1S[j] = T1[0] * Sf[j] + T1[1] * Sf[3 + j] + T1[2] * Sf[6 + j];
    }
    double dS[9];  // gradient w.r.t. Sigma3 as a general matrix
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) dS[3 * i + j] = da * T0[i] * T0[j] + db * T0[i] * T1[j] + dc * T1[i] * T1[j];
    double dT0[3], dT1[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        dT0[j] = 2.0 * da * T0S[j] + db * T1S[j];
        dT1[j] = db * T0S[j] + 2.0 * dc * T1S[j];
    }
    // Tm = J R: row 0 = J00 R0 + J02 R2, row 1 = J11 R1 + J12 R2
    double R[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) R[q] = V.R[q];
    const double dJ00 = dT0[0] * R[0] + dT0[1] * R[1] + dT0[2] * R[2];
    const double dJ02 = dT0[0] * R[6] + dT0[1] * R[7] + dT0[2] * R[8];
    const double dJ11 = dT1[0] * R[3] + dT1[1] * R[4] + dT1[2] * R[5];
    const double dJ12 = dT1[0] * R[6] + dT1[1] * R[7] + dT1[2] * R[8];
    const double x = P.pc[0], y = P.pc[1], z = P.pc[2];
    const double iz = 1.0 / z, iz2 = iz * iz, iz3 = iz2 * iz;
    const double fx = V.fx, fy = V.fy;
    double dp[3];
    dp[0] = dJ02 * (-fx * iz2) + du * fx * iz;
    dp[1] = dJ12 * (-fy * iz2) + dv * fy * iz;
    dp[2] = dJ00 * (-fx * iz2) + dJ02 * (2.0 * fx * x * iz3) + dJ11 * (-fy * iz2) + dJ12 * (2.0 * fy * y * iz3) -
            du * fx * x * iz2 - dv * fy * y * iz2;
#pragma unroll
    for (int m = 0; m < 3; ++m) dmu[m] += R[m] * dp[0] + R[3 + m] * dp[1] + R[6 + m] * dp[2];

    // Sigma3 = M M^T, M = Rq diag(s)
    double Rq[9];
    quat_rot(P.q, Rq);
    double M[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) M[3 * r + cc] = Rq[3 * r + cc] * P.s[cc];
    double ds[3] = {0.0, 0.0, 0.0}, dR[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) acc += (dS[3 * i + q] + dS[3 * q + i]) * M[3 * q + j];
            ds[j] += acc * Rq[3 * i + j];
            dR[3 * i + j] = acc * P.s[j];
        }
    const double qw = P.q[0], qx = P.q[1], qy = P.q[2], qz = P.q[3];
    double dq[4];
    dq[0] = 2.0 * (-qz * dR[1] + qy * dR[2] + qz * dR[3] - qx * dR[5] - qy * dR[6] + qx * dR[7]);
    dq[1] = 2.0 * (qy * dR[1] + qz * dR[2] + qy * dR[3] - 2.0 * qx * dR[4] - qw * dR[5] + qz * dR[6] + qw * dR[7] -
                   2.0 * qx * dR[8]);
    dq[2] = 2.0 * (-2.0 * qy * dR[0] + qx * dR[1] + qw * dR[2] + qx * dR[3] + qz * dR[5] - qw * dR[6] + qz * dR[7] -
                   2.0 * qy * dR[8]);
    dq[3] = 2.0 * (-2.0 * qz * dR[0] - qw * dR[1] + qx * dR[2] + qw * dR[3] - 2.0 * qz * dR[4] + qy * dR[5] +
                   qx * dR[6] + qy * dR[7]);
    const double qd = qw * dq[0] + qx * dq[1] + qy * dq[2] + qz * dq[3];
    double dqr[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) dqr[m] = (dq[m] - P.q[m] * qd) / P.qlen;

    // gradient with respect to the interpolated attributes; the gather
    // weights it by (1 - t) for the node and t for the parent
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        row[m] = (float)dmu[m];
        row[3 + m] = (float)ds[m];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) row[6 + m] = (float)dqr[m];
    if (use_par) {
        const float3 mn = *reinterpret_cast<const float3 *>(h.mean + 3 * (size_t)node);
        const float3 mp = *reinterpret_cast<const float3 *>(h.mean + 3 * (size_t)par);
        const float3 sn = *reinterpret_cast<const float3 *>(h.scale + 3 * (size_t)node);
        const float3 sp = *reinterpret_cast<const float3 *>(h.scale + 3 * (size_t)par);
        const float4 qn = *reinterpret_cast<const float4 *>(h.rot + 4 * (size_t)node);
        const float4 qp = *reinterpret_cast<const float4 *>(h.rot + 4 * (size_t)par);
        dt += dmu[0] * ((double)mp.x - (double)mn.x) + dmu[1] * ((double)mp.y - (double)mn.y) +
              dmu[2] * ((double)mp.z - (double)mn.z);
        dt += ds[0] * ((double)sp.x - (double)sn.x) + ds[1] * ((double)sp.y - (double)sn.y) +
              ds[2] * ((double)sp.z - (double)sn.z);
        dt += dqr[0] * ((double)qp.x - (double)qn.x) + dqr[1] * ((double)qp.y - (double)qn.y) +
              dqr[2] * ((double)qp.z - (double)qn.z) + dqr[3] * ((double)qp.w - (double)qn.w);
    }
    // opacity through |o|
    row[10] = (float)((P.on_raw > 0.0 ? 1.0 : (P.on_raw < 0.0 ? -1.0 : 0.0)) * don);
    row[11] = (float)((P.op_raw > 0.0 ? 1.0 : (P.op_raw < 0.0 ? -1.0 : 0.0)) * dop);
    row[kPG - 1] = 0.0f;
    dt_out = use_par ? (float)dt : 0.0f;
}

// Takes the chunks of cut entries in the forward's order and writes, for the
// visible ones that reached a pixel (more than a third at 32 views far into a
// scene did not: their screen-gradient row is all zeros), the attribute-
// gradient rows at their cut positions; live: one bit per cut entry, the rows
// that the gather has to read.  With g_dt, dL/dt of all others is
// cleared.  A wave's screen-gradient rows lie one behind the other (visible
// entries rank in cut order), and so do its colour Jacobians and the rows it
// writes: all three pass through the wave's LDS in whole lines, the loads
// under way while the entries are projected.  2.63 -> 2.11 ms at 30 M visible
// splats of 32 views, 572 -> 444 us at 8 views of a 3 M node hierarchy (of it
// 0.13 ms and 46 us are the order's); what bounds it now is half memory (a
// 96-byte row, a 48-byte Jacobian and the parameters read, 80 bytes written)
// and half FP64 arithmetic at 3 waves per SIMD.  Listing the entries whose row
// is not all zero first (64% of them) was slower: 3.2 ms, the list is a longer
// chain than the work saved.
__global__ __launch_bounds__(kT, 3) void k_preprocess_bwd(DevHier h, const DevView *__restrict__ views, int nv,
                                                       const uint32_t *__restrict__ cut_base,
                                                       const int32_t *__restrict__ cut_ids,
                                                       const double *__restrict__ cut_t,
                                                       const uint32_t *__restrict__ cut_total, uint32_t cap,
                                                       const uint64_t *__restrict__ vis_mask,
                                                       const uint64_t *__restrict__ pos_mask,
                                                       const float *__restrict__ cjac,
                                                       const uint32_t *__restrict__ vis_offsets,
                                                       const uint32_t *__restrict__ order,
                                                       const double *__restrict__ sgrad, float *__restrict__ pg,
                                                       uint64_t *__restrict__ live, float *__restrict__ g_dt)
{
    // per wave: 64 rows of 96 B (screen gradients) and 64 of 48 B (Jacobians);
    // the 64 rows of 80 B written take the place of the former
    constexpr int kRows = 64 * 96, kStage = kRows + 64 * 48;
    static_assert(64 * kPG * 4 <= kRows, "the written rows fit");
    __shared__ __align__(16) char s_stage[kT / 64][kStage];
    const uint32_t total = min(*cut_total, cap), nchunks = (total + kT - 1) / kT;
    const uint32_t at = order ? chunk_place(blockIdx.x) : blockIdx.x;
    if (at >= nchunks) return;
    const uint32_t chunk = order ? order[at] : at;
    const uint32_t k = chunk * kT + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t rank = vis_offsets[chunk];  // of the wave's first visible entry
    uint64_t m = 0ull;                   // its visible entries
#pragma unroll
    for (int q = 0; q < kT / 64; ++q) {
        const uint64_t mq = vis_mask[chunk * (kT / 64) + q];
        if (q < w) rank += (uint32_t)__popcll(mq);
        if (q == w) m = mq;
    }
    m = (uint64_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)m) & 0xFFFFFFFFull |
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(m >> 32)) << 32;
    const bool seen = (m >> lane) & 1ull;
    if (g_dt && !seen && k < total) g_dt[k] = 0.0f;
    if (m == 0ull) {
        if (lane == 0) live[k >> 6] = 0ull;
        return;
    }
    char *stage = s_stage[w];
    const uint32_t cnt = (uint32_t)__popcll(m), kw = k & ~63u;
    const float *rows = reinterpret_cast<const float *>(sgrad + (size_t)rank * 12);
    const float *jac = cjac + (size_t)kw * 12;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const uint32_t e = 64u * i + (uint32_t)lane;
        if (e < 6u * cnt) load_lds16(rows + 4 * e, stage + 1024 * i);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t e = 64u * i + (uint32_t)lane;
        if ((m >> (e / 3u)) & 1ull) load_lds16(jac + 4 * e, stage + kRows + 1024 * i);
    }
    float row[kPG];
#pragma unroll
    for (int q = 0; q < kPG; ++q) row[q] = 0.0f;
    bool any = false;
    if (seen) {
        float dt = 0.0f;
        const uint32_t r = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        entry_bwd(h, views[view_of_wave(cut_base, nv, k)], k, (uint32_t)cut_ids[k], cut_t[k],
                  pos_mask + (size_t)(k >> 6) * 3, reinterpret_cast<const double *>(stage + 96 * r),
                  reinterpret_cast<const float *>(stage + kRows + 48 * lane), row, any, dt);
        if (g_dt) g_dt[k] = dt;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    wave_lds_sync();
    float4 *o = reinterpret_cast<float4 *>(stage);
    if (seen)
#pragma unroll
        for (int q = 0; q < kPG / 4; ++q)
            o[kPG / 4 * lane + q] = make_float4(row[4 * q], row[4 * q + 1], row[4 * q + 2], row[4 * q + 3]);
    wave_lds_sync();
    const uint64_t lm = __ballot(any);
    if (lane == 0) live[k >> 6] = lm;
    store_rows<kPG / 4>(o, reinterpret_cast<float4 *>(pg + (size_t)kw * kPG), lm, lane);
}

// Per view and mask word, the nodes whose cut entry has an attribute-gradient
// row (sel): the entries' bits live[...] of the word's run in the cut, spread
// to the places of the selected nodes.  A workgroup takes 64 words of 8 views,
// one wave per view, and also notes which of the views have a node in a word:
// word_views holds, for every 64 views, 64 bits per word.  Streams its bits:
// 0.45 GB in 0.146 ms at 44.5 M nodes and 32 views.
constexpr int kLiveViews = 8;

__global__ __launch_bounds__(64 * kLiveViews) void k_live_nodes(
    const uint64_t *__restrict__ masks, const uint32_t *__restrict__ word_off, int64_t words, int nv,
    const uint64_t *__restrict__ live, const uint32_t *__restrict__ cut_total, uint32_t cap,
    uint64_t *__restrict__ sel, uint8_t *__restrict__ word_views)
{
    __shared__ uint64_t s_has[kLiveViews];  // per view, its words with a node
    const int lane = threadIdx.x & 63, u = threadIdx.x >> 6, v = blockIdx.y * kLiveViews + u;
    const int64_t w = (int64_t)blockIdx.x * 64 + lane;
    uint64_t r = 0ull;
    if (w < words && v < nv) {
        const int64_t i = (int64_t)v * words + w;
        const uint64_t m = masks[i];
        if (m) {
            const uint32_t total = min(*cut_total, cap), p = word_off[i], sh = p & 63u;
            const uint32_t n = p < total ? min((uint32_t)__popcll(m), total - p) : 0u;
            uint64_t b = 0ull;  // the run's bits
            if (n) b = live[p >> 6] >> sh;
            if (sh + n > 64u) b |= live[(p >> 6) + 1] << (64u - sh);
            if (n < 64u) b &= (1ull << n) - 1ull;
            if (n == 64u) r = b;
            else
                for (uint64_t k = m; b; b >>= 1, k &= k - 1ull)
                    if (b & 1ull) r |= k & (~k + 1ull);
        }
        sel[i] = r;
    }
    const uint64_t h = __ballot(r != 0ull);
    if (lane == 0) s_has[u] = h;
    __syncthreads();
    if (u == 0 && w < words) {
        uint32_t views = 0;
#pragma unroll
        for (int q = 0; q < kLiveViews; ++q) views |= (uint32_t)((s_has[q] >> lane) & 1ull) << q;
        const int64_t row = w * (8 * ((nv + 63) / 64));
        word_views[row + blockIdx.y] = (uint8_t)views;
        if (blockIdx.y + 1 == gridDim.y)  // the last views' workgroup clears the bits behind them
            for (int g = gridDim.y; g < 8 * ((nv + 63) / 64); ++g) word_views[row + g] = 0;
    }
}

// Gathers each interior node's parameter gradient from the cut entries of
// every view: its own entry weighted 1 - t, and the entry of each child in
// the cut with t > 0 weighted by that child's t (leaves are frozen; both
// opacity terms enter alpha directly, unweighted).  One thread per interior
// node, views and entries in a fixed order: no atomics, and the result is
// reproducible bit for bit.  Positions come from the cut's bit masks: node j
// of view v sits at word_off[v][j / 64] plus the selected nodes below j in
// its word.  The children of a node are contiguous ids, so one or two mask
// words give all of them at once.
//
// Bound by the chain of dependent loads (words of a view, then rows) at the 12
// waves per CU that the 59 sums and two rows leave.  A wave goes through the
// views together, and only through those that have an entry with a row in one
// of its words (word_views), two rows in flight: 3.45 -> 1.56 ms for 14.5 M
// interior nodes and 32 views, 495 -> 327 us for 1 M and 8 views.  Each thread through views of its own, reading masks,
// tile counts and t of every entry, took the former; listing the entries first,
// or 16 waves per CU with 40 spilled registers, 5.3 ms.
//
// FUSED: instead of adding the sum to the gradient arrays, the thread
// applies the optimiser step to its node right away (every interior node,
// those with no contribution too, whose gradient is zero): the gradient is
// never written, re-read or cleared.

// The fused optimiser step of one block: thread t holds the gathered
// gradient of interior node q0 + t (node id `node`; zero past the end).  The
// mean and scale rows (3 floats each) and the SH rows (48 floats, 64 rows at
// a time) go through LDS, so that the update walks the moments contiguously
// and each parameter row with consecutive lanes, as the separate step does;
// rotation (one 16-byte row) and opacity are stepped by the row's own
// thread from its registers.  The separate step reads 0 + sum
// from a cleared gradient array; the same value is formed here (it turns -0
// into +0), and the arithmetic is the same function, so both agree bit for
// bit.  Every thread of the block calls it (barriers).
constexpr int kAdamLds = 64 * 48;  // floats of the staging buffer (>= kT x 11)
static_assert(kT * 11 <= kAdamLds && kT % 64 == 0, "staging buffer");

__device__ __forceinline__ void adam_block(const AdamRows &ad, int64_t n_interior, int64_t q0, int32_t node,
                                           const float (&a)[11], const float (&ash)[48])
{
    __shared__ float s_g[kAdamLds];
    __shared__ int32_t s_node[kT];  // the block's node ids
    const int t = threadIdx.x;
    const int rows = (int)min<int64_t>(kT, n_interior - q0);  // >= 1: the block holds an interior node
    s_node[t] = node;
#pragma unroll
    for (int k = 0; k < 11; ++k) s_g[11 * t + k] = a[k];
    __syncthreads();
    // mean and scale: 3 floats per row
#pragma unroll
    for (int grp = 0; grp < 2; ++grp) {
        const AdamScalars s = ad.sc[grp];
        float *p = ad.p[grp], *m = ad.m[grp] + 3 * q0, *v = ad.v[grp] + 3 * q0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int e = t + kT * k, r = e / 3, c = e - 3 * r;
            if (r < rows) {
                const int64_t pi = 3 * (int64_t)s_node[r] + c;
                float pk = p[pi], mk = m[e], vk = v[e];
                adam_one(pk, 0.0f + s_g[11 * r + 3 * grp + c], mk, vk, s);
                p[pi] = pk;
                m[e] = mk;
                v[e] = vk;
            }
        }
    }
    if (t < rows) {
        // rotation: one 16-byte row per thread; opacity: one float
        const AdamScalars s = ad.sc[2];
        float4 *p4 = reinterpret_cast<float4 *>(ad.p[2]) + node, *m4 = reinterpret_cast<float4 *>(ad.m[2]) + q0 + t,
               *v4 = reinterpret_cast<float4 *>(ad.v[2]) + q0 + t;
        float4 pk = *p4, mk = *m4, vk = *v4;
        adam_one(pk.x, 0.0f + a[6], mk.x, vk.x, s);
        adam_one(pk.y, 0.0f + a[7], mk.y, vk.y, s);
        adam_one(pk.z, 0.0f + a[8], mk.z, vk.z, s);
        adam_one(pk.w, 0.0f + a[9], mk.w, vk.w, s);
        *p4 = pk;
        *m4 = mk;
        *v4 = vk;
        const AdamScalars so = ad.sc[3];
        float po = ad.p[3][node], mo = ad.m[3][q0 + t], vo = ad.v[3][q0 + t];
        adam_one(po, 0.0f + a[10], mo, vo, so);
        ad.p[3][node] = po;
        ad.m[3][q0 + t] = mo;
        ad.v[3][q0 + t] = vo;
    }
    // SH: 64 rows of 12 float4 at a time
    const AdamScalars s = ad.sc[4];
    float4 *p4 = reinterpret_cast<float4 *>(ad.p[4]);
    float4 *m4 = reinterpret_cast<float4 *>(ad.m[4]) + 12 * q0, *v4 = reinterpret_cast<float4 *>(ad.v[4]) + 12 * q0;
    float4 *g4 = reinterpret_cast<float4 *>(s_g);
#pragma unroll 1
    for (int r0 = 0; r0 < rows; r0 += 64) {
        __syncthreads();  // the previous contents read
        if (t >= r0 && t < r0 + 64)
#pragma unroll
            for (int k = 0; k < 12; ++k)
                g4[12 * (t - r0) + k] = make_float4(ash[4 * k], ash[4 * k + 1], ash[4 * k + 2], ash[4 * k + 3]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int e = t + kT * k, r = e / 12, c = e - 12 * r;  // row r0 + r, vector c
            if (r0 + r < rows) {
                const int64_t pi = 12 * (int64_t)s_node[r0 + r] + c;
                const int64_t mi = 12 * (int64_t)r0 + e;
                const float4 g = g4[e];
                float4 pk = p4[pi], mk = m4[mi], vk = v4[mi];
                adam_one(pk.x, 0.0f + g.x, mk.x, vk.x, s);
                adam_one(pk.y, 0.0f + g.y, mk.y, vk.y, s);
                adam_one(pk.z, 0.0f + g.z, mk.z, vk.z, s);
                adam_one(pk.w, 0.0f + g.w, mk.w, vk.w, s);
                p4[pi] = pk;
                m4[mi] = mk;
                v4[mi] = vk;
            }
        }
    }
}

template <bool FUSED>
__global__ __launch_bounds__(kT, 3) void k_grad_gather(DevHier h, int nv, const uint64_t *__restrict__ masks,
                                                    int64_t words, const uint32_t *__restrict__ word_off,
                                                    const uint64_t *__restrict__ sel,
                                                    const uint64_t *__restrict__ word_views,
                                                    const float *__restrict__ pg,
                                                    const int32_t *__restrict__ interior, int64_t n_interior,
                                                    float *__restrict__ g_mean, float *__restrict__ g_scale,
                                                    float *__restrict__ g_rot, float *__restrict__ g_op,
                                                    float *__restrict__ g_sh, AdamRows ad)
{
    const int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x;
    const bool valid = q < n_interior;  // the fused step's threads past the end still help in its update
    if (!FUSED && !valid) return;
    const int64_t i = valid ? interior[q] : 0;
    float a[11];  // mean 3, scale 3, rotation 4, opacity
    float ash[48];
#pragma unroll
    for (int m = 0; m < 11; ++m) a[m] = 0.0f;
#pragma unroll
    for (int m = 0; m < 48; ++m) ash[m] = 0.0f;
    bool any = false;
    if (valid) {
        const int64_t c0 = h.child_begin[i], c1 = c0 + h.child_count[i];  // children [c0, c1)
        // adds the attribute gradient of a contributing entry (row r), weighted
        // 1 - t as the node's own entry (op 10: node opacity term) or t as a
        // child's entry (op 11: parent opacity term)
        auto add = [&](const float4 (&r)[5], int op) {
            const float t = r[4].z, w = op == 10 ? 1.0f - t : t;
            if (op == 11 && !(t > 0.0f)) return;
            const float g[15] = {r[0].x, r[0].y, r[0].z, r[0].w, r[1].x, r[1].y, r[1].z, r[1].w,
                                 r[2].x, r[2].y, r[2].z, r[2].w, r[3].x, r[3].y, r[3].z};
#pragma unroll
            for (int m = 0; m < 10; ++m) a[m] += w * g[m];
            a[10] += op == 10 ? g[10] : g[11];
            float Y[16];  // the SH basis of the entry's direction, in FP32 as the forward evaluated it
            sh_eval_f(r[3].w, r[4].x, r[4].y, Y);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float wc = w * g[12 + c];
#pragma unroll
                for (int k = 0; k < 16; ++k) ash[3 * k + c] += wc * Y[k];
            }
            any = true;
        };
        const int64_t wi = i >> 6, wa = c0 >> 6, wb = (c1 - 1) >> 6;
        const uint64_t below_i = (1ull << (i & 63)) - 1ull, own_bit = 1ull << (i & 63);
        // the children's bits in their first word (wa) and last word (wb)
        const int lo = (int)(c0 & 63), hi = (int)((c1 - 1) & 63);
        const uint64_t k_lo = ~((1ull << lo) - 1ull), k_hi = hi == 63 ? ~0ull : ((1ull << (hi + 1)) - 1ull);
        const int groups = (nv + 63) / 64;
#pragma unroll 1
        for (int g = 0; g < groups; ++g) {
            // the views with an entry in a word of the node or its children,
            // one after the other, the threads of the wave together
            uint64_t hit = word_views[wi * groups + g];
            for (int64_t w = wa; w <= wb; ++w) hit |= word_views[w * groups + g];
            uint32_t h0 = (uint32_t)hit, h1 = (uint32_t)(hit >> 32);
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                h0 |= (uint32_t)__shfl_xor((int)h0, d, 64);
                h1 |= (uint32_t)__shfl_xor((int)h1, d, 64);
            }
            uint64_t all = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)h1) << 32 |
                           (uint32_t)__builtin_amdgcn_readfirstlane((int)h0);
#pragma unroll 1
            for (; all; all &= all - 1ull) {
                const int v = 64 * g + __builtin_ctzll(all);
                const bool h = (hit >> (v & 63)) & 1ull;
                const int64_t at = (int64_t)v * words;
                const uint64_t *sv = sel + at, *mv = masks + at;
                const uint32_t *ov = word_off + at;
                bool own = false;
                uint32_t po = 0;
                if (h) {
                    const uint64_t so = sv[wi], mo = mv[wi];
                    own = (so & own_bit) != 0ull;
                    po = ov[wi] + (uint32_t)__popcll(mo & below_i);
                }
                int64_t w = h ? wa : wb + 1;
                do {  // two words of children at a time (most nodes: all of them)
                    uint64_t ca = 0ull, cb = 0ull, ma = 0ull, mb = 0ull;
                    uint32_t pa = 0, pb = 0;
                    if (w <= wb) {
                        ca = sv[w] & (w == wa ? k_lo : ~0ull) & (w == wb ? k_hi : ~0ull);
                        ma = mv[w];
                        pa = ov[w];
                    }
                    if (w < wb) {
                        cb = sv[w + 1] & (w + 1 == wb ? k_hi : ~0ull);
                        mb = mv[w + 1];
                        pb = ov[w + 1];
                    }
                    w += 2;
                    auto child = [&](uint32_t &pos) -> bool {
                        const bool first = ca != 0ull;
                        const uint64_t c = first ? ca : cb, b = c & (~c + 1ull);
                        pos = (first ? pa : pb) + (uint32_t)__popcll((first ? ma : mb) & (b - 1ull));
                        ca &= first ? ~b : 0ull;
                        cb &= first ? ~0ull : ~b;
                        return c != 0ull;
                    };
                    for (;;) {  // two rows in flight: the node's own, then its children's
                        uint32_t p0 = po, p1;
                        const bool o0 = own, b0 = own || child(p0);
                        own = false;
                        if (!__any(b0)) break;
                        const bool b1 = child(p1);
                        float4 r0[5], r1[5];
                        if (b0) {
                            const float4 *g4 = reinterpret_cast<const float4 *>(pg + (size_t)p0 * kPG);
#pragma unroll
                            for (int q = 0; q < 5; ++q) r0[q] = g4[q];
                        }
                        if (b1) {
                            const float4 *g4 = reinterpret_cast<const float4 *>(pg + (size_t)p1 * kPG);
#pragma unroll
                            for (int q = 0; q < 5; ++q) r1[q] = g4[q];
                        }
                        if (b0) add(r0, o0 ? 10 : 11);
                        if (b1) add(r1, 11);
                    }
                } while (__any(w <= wb));
            }
        }
    }
    if constexpr (FUSED) {
        adam_block(ad, n_interior, (int64_t)blockIdx.x * kT, (int32_t)i, a, ash);
        return;
    }
    if (!any) return;
    // node-major records: vector read-modify-write
    float3 *gm = reinterpret_cast<float3 *>(g_mean + 3 * i), *gs = reinterpret_cast<float3 *>(g_scale + 3 * i);
    float4 *gr = reinterpret_cast<float4 *>(g_rot + 4 * i), *gh = reinterpret_cast<float4 *>(g_sh + 48 * i);
    float3 m3 = *gm, s3 = *gs;
    float4 r4 = *gr;
    m3.x += a[0];
    m3.y += a[1];
    m3.z += a[2];
    s3.x += a[3];
    s3.y += a[4];
    s3.z += a[5];
    r4.x += a[6];
    r4.y += a[7];
    r4.z += a[8];
    r4.w += a[9];
    *gm = m3;
    *gs = s3;
    *gr = r4;
    g_op[i] += a[10];
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        float4 h4 = gh[q];
        h4.x += ash[4 * q];
        h4.y += ash[4 * q + 1];
        h4.z += ash[4 * q + 2];
        h4.w += ash[4 * q + 3];
        gh[q] = h4;
    }
}

}  // namespace

void launch_chunk_order(const uint32_t *block_offsets, int nblocks, int nv, const uint32_t *cut_total,
                        uint32_t *order, uint32_t cap, hipStream_t st)
{
    const int runs = (nblocks + kOrderBlocks - 1) / kOrderBlocks, per = kT / 64;
    hipLaunchKernelGGL(k_chunk_order, dim3((uint32_t)((runs + per - 1) / per)), dim3(kT), 0, st, block_offsets,
                       nblocks, nv, cut_total, order, (cap + kT - 1) / kT);
}

void launch_preprocess(const DevHier &h, const DevView *views, int nv, const uint32_t *cut_base,
                       const int32_t *cut_ids, const double *cut_t, const uint32_t *cut_total, uint32_t cap,
                       SplatRec *recs, double4 *axes, uint32_t *depth_key, uint4 *trec,
                       float *cjac, uint64_t *vis_mask, uint64_t *pos_mask, uint32_t *vis_block_counts,
                       const uint32_t *order, int tile_w, int tile_h, uint32_t *inf_colour, hipStream_t st)
{
    uint32_t blocks = (cap + kT - 1) / kT;
    if (!blocks) return;
    if (order) blocks = chunk_grid(blocks);
    auto k = (uintptr_t)h.sh % 16 == 0 ? k_preprocess<true> : k_preprocess<false>;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kT), 0, st, h, views, nv, cut_base, cut_ids, cut_t, cut_total,
                       cap, recs, axes, depth_key, trec, cjac, vis_mask, pos_mask, vis_block_counts, order, tile_w,
                       tile_h, inf_colour);
}

void launch_compact_visible(const uint64_t *vis_mask, const uint32_t *vis_block_offsets, const uint32_t *cut_total,
                            uint32_t cap, const uint32_t *depth_key, uint32_t *keys, uint32_t *vals,
                            uint32_t *vis_rank, hipStream_t st)
{
    const uint32_t blocks = (cap + kT - 1) / kT;
    if (!blocks) return;
    hipLaunchKernelGGL(k_compact_visible, dim3(blocks), dim3(kT), 0, st, vis_mask, vis_block_offsets, cut_total, cap,
                       depth_key, keys, vals, vis_rank);
}

void launch_zero_rows(double *rows, int width, const uint32_t *vis_total, uint32_t vis_cap, hipStream_t st)
{
    const uint64_t need = ((uint64_t)vis_cap * width + kT - 1) / kT;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(need, 8192);
    if (!blocks) return;
    hipLaunchKernelGGL(k_zero_rows, dim3(blocks), dim3(kT), 0, st, rows, width, vis_total, vis_cap);
}

void launch_plan_depth(const uint32_t *cut_base, int nv, const uint64_t *vis_mask, const uint32_t *vis_offsets,
                       const uint32_t *cut_total, uint32_t cap, const uint32_t *vis_total, uint32_t *vis_bounds,
                       const SortScratch &s, hipStream_t st)
{
    hipLaunchKernelGGL(k_plan_depth, dim3(1), dim3(kMaxViews), 0, st, cut_base, nv, vis_mask, vis_offsets, cut_total,
                       cap, vis_total, vis_bounds, s.plan, sort_grid(cap, nv), s.tot, sort_totals(32, nv));
}

void launch_plan_pairs(const uint32_t *vis_bounds, const DevView *views, int nv, const uint32_t *pair_offsets,
                       const uint32_t *vis_total, uint32_t vis_cap, const uint32_t *pair_total, uint32_t pair_cap,
                       int bits, const SortScratch &s, hipStream_t st)
{
    hipLaunchKernelGGL(k_plan_pairs, dim3(1), dim3(kMaxViews), 0, st, vis_bounds, views, nv, pair_offsets, vis_total,
                       vis_cap, pair_total, pair_cap, s.plan, sort_grid(pair_cap, nv), s.tot, sort_totals(bits, nv));
}

void launch_gather_tiles(const uint4 *trec, const uint32_t *sorted_vals, const uint32_t *vis_total, uint32_t vis_cap,
                         uint32_t *counts, uint2 *rect, uint32_t *jrank, hipStream_t st)
{
    const uint32_t blocks = (vis_cap + kT - 1) / kT;
    if (!blocks) return;
    hipLaunchKernelGGL(k_gather_tiles, dim3(blocks), dim3(kT), 0, st, trec, sorted_vals, vis_total, vis_cap, counts,
                       rect, jrank);
}

void launch_det_sum(const double *part, const uint32_t *pair_offsets, const uint32_t *sorted_vals,
                    const uint32_t *vis_rank, const uint32_t *vis_total, uint32_t vis_cap,
                    const uint32_t *pair_total, uint32_t pair_cap, double *sgrad, hipStream_t st)
{
    const uint32_t blocks = (vis_cap + kT - 1) / kT;
    if (!blocks) return;
    hipLaunchKernelGGL(k_det_sum, dim3(blocks), dim3(kT), 0, st, part, pair_offsets, sorted_vals, vis_rank, vis_total,
                       vis_cap, pair_total, pair_cap, sgrad);
}

void launch_duplicate(const uint2 *rect, const DevView *views, int nv, const uint32_t *cut_base,
                      const uint32_t *sorted_vals, const uint32_t *pair_offsets, const uint32_t *block_first,
                      const uint32_t *vis_total, uint32_t vis_cap, const uint32_t *pair_total, uint32_t pair_cap,
                      uint32_t *pair_keys, uint32_t *pair_vals, Counters *ctr, hipStream_t st)
{
    const uint32_t dblocks = (pair_cap + kDupPairs - 1) / kDupPairs;
    if (!dblocks) return;
    hipLaunchKernelGGL(k_duplicate, dim3(dblocks), dim3(kT), 0, st, rect, views, nv, cut_base, sorted_vals,
                       pair_offsets, block_first, vis_total, vis_cap, pair_total, pair_cap, pair_keys, pair_vals, ctr);
}

uint32_t duplicate_blocks(uint32_t pair_cap)
{
    return (pair_cap + kDupPairs - 1) / kDupPairs;
}

void launch_ranges(const uint32_t *pair_keys, const uint32_t *pair_total, uint32_t pair_cap, uint2 *ranges,
                   hipStream_t st)
{
    const uint32_t blocks = (uint32_t)(((uint64_t)pair_cap + kT * kRangeItems - 1) / (kT * kRangeItems));
    if (!blocks) return;
    hipLaunchKernelGGL(k_ranges, dim3(blocks), dim3(kT), 0, st, pair_keys, pair_total, pair_cap, ranges);
}

void launch_init(Counters *ctr, uint32_t *tile_hist, uint2 *ranges, uint32_t n_tiles, hipStream_t st)
{
    const uint32_t blocks = std::min<uint32_t>(std::max<uint32_t>((n_tiles + kT - 1) / kT, 1u), 2048u);
    hipLaunchKernelGGL(k_init, dim3(blocks), dim3(kT), 0, st, (uint32_t *)ctr, (uint32_t)(sizeof(Counters) / 4),
                       tile_hist, 2u * kTileBins, ranges, n_tiles);
}

void launch_tile_order(const uint2 *ranges, uint32_t n_tiles, uint32_t *tile_hist, uint32_t *order, hipStream_t st)
{
    if (!n_tiles) return;
    const uint32_t blocks = (n_tiles + kTileBlock - 1) / kTileBlock;
    hipLaunchKernelGGL(k_tile_bins, dim3(blocks), dim3(kT), 0, st, ranges, n_tiles, tile_hist);
    hipLaunchKernelGGL(k_tile_place, dim3(blocks), dim3(kT), 0, st, ranges, n_tiles, tile_hist, tile_hist + kTileBins,
                       order);
}

void launch_fill_u32(uint32_t *p, uint32_t value, size_t n, hipStream_t st)
{
    if (!n) return;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, value, n);
}

void launch_preprocess_backward(const DevHier &h, const DevView *views, int nv, const uint32_t *cut_base,
                                const int32_t *cut_ids, const double *cut_t, const uint32_t *cut_total, uint32_t cap,
                                const uint64_t *vis_mask, const uint64_t *pos_mask, const float *cjac,
                                const uint32_t *vis_offsets,
                                const uint32_t *order, const double *sgrad, float *pg, uint64_t *live,
                                uint64_t *sel, uint64_t *word_views, const uint64_t *masks, int64_t words, const uint32_t *word_off,
                                const int32_t *interior, int64_t n_interior,
                                float *g_mean, float *g_scale, float *g_rot, float *g_opacity, float *g_sh,
                                float *g_dt, const AdamRows *fused, hipStream_t st)
{
    uint32_t blocks = (cap + kT - 1) / kT;
    if (!blocks) return;
    if (order) blocks = chunk_grid(blocks);
    hipLaunchKernelGGL(k_preprocess_bwd, dim3(blocks), dim3(kT), 0, st, h, views, nv, cut_base, cut_ids, cut_t,
                       cut_total, cap, vis_mask, pos_mask, cjac, vis_offsets, order, sgrad, pg, live, g_dt);
    const int64_t gblocks = (n_interior + kT - 1) / kT;
    if (!gblocks) return;
    hipLaunchKernelGGL(k_live_nodes, dim3((uint32_t)((words + 63) / 64), (nv + kLiveViews - 1) / kLiveViews),
                       dim3(64 * kLiveViews), 0, st,
                       masks, word_off, words, nv, live, cut_total, cap, sel, reinterpret_cast<uint8_t *>(word_views));
    if (fused)
        hipLaunchKernelGGL(k_grad_gather<true>, dim3((uint32_t)gblocks), dim3(kT), 0, st, h, nv, masks, words,
                           word_off, sel, word_views, pg, interior, n_interior, nullptr, nullptr,
                           nullptr, nullptr, nullptr, *fused);
    else
        hipLaunchKernelGGL(k_grad_gather<false>, dim3((uint32_t)gblocks), dim3(kT), 0, st, h, nv, masks, words,
                           word_off, sel, word_views, pg, interior, n_interior, g_mean, g_scale, g_rot,
                           g_opacity, g_sh, AdamRows{});
}

}  // namespace hgs
