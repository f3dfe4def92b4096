// Per-tile alpha blending (forward) and its backward.
//
// One workgroup per tile of TW x TH pixels; each 64-lane wave owns an 8x8
// sub-tile, one lane per pixel, and each row of 16 lanes one 4x4 quarter of
// it.  The tile's splats (sorted front to back) are staged through LDS in
// batches of one record per thread, each with one bit per quarter telling
// whether any pixel of the quarter can reach alpha = 1/255.  Every quarter
// walks a list of the splats it may take only (a small splat touches one or
// two of them), so that the four quarters of a wave step through different
// splats together.  Per pixel and splat (Sec. 3 Eq. (alpha) with the
// projected Gaussian G; Eq. (alphap) generalised to K children, Sec. 5.2;
// the weight t of Eq. (t_interp) as the parent's weight; clamp of Sec. 7.3):
//   G     = exp(-q/2),  q = d^T conic d  (d = pixel centre - mean), evaluated
//           as exp2(-(u1^2 + u2^2)) with u_i = w_i . d on the conic's scaled
//           eigen-axes (see SplatRec)
//   a_n   = min(0.99, A_n G),  a_p = min(0.99, A_p G)
//   alpha = (1 - t) a_n + t (1 - (1 - a_p)^(1/K))     (= a_n when t = 0)
//   skip when alpha < 1/255; stop before T (1 - alpha) < 1e-4;
//   C += c alpha T;  T *= 1 - alpha.
// The backward walks each tile back to front from the final transmittance
// and the index of the last contributor of each pixel, recovering the
// transmittance in front of every splat by dividing by (1 - alpha) (no
// per-pixel lists), reduces each splat's gradient over the pixels of a quarter
// by lane exchanges and over the quarters of the tile in LDS (FP64 atomics), and
// adds it once per tile, in FP64, to the splat's screen-space gradient.
#include <algorithm>
#include <cstddef>
#include <map>
#include <mutex>

#include "hgs_internal.h"

namespace hgs {

namespace {

// Staged splat, per 8x8 block of the tile: c = w . (block corner + 1/2 - mean)
// in FP64, so that a lane only adds w . (its offset inside the block): the
// result depends on the pixel alone, not on the tile size.
__device__ __forceinline__ void block_offsets(const SplatRec &r, const double4 &W, int bx, int by, float &c1,
                                              float &c2, float &dx0, float &dy0)
{
#pragma clang fp contract(off)
    const double dx = ((double)(bx - r.ax) + 0.5) - (double)r.fx;
    const double dy = ((double)(by - r.ay) + 0.5) - (double)r.fy;
    c1 = (float)(dx * W.x + dy * W.y);
    c2 = (float)(dx * W.z + dy * W.w);
    dx0 = (float)dx;
    dy0 = (float)dy;
}

// Identical arithmetic in forward and backward (explicit FMAs, no other
// contraction), so that the backward reproduces the forward's decisions bit
// for bit.
__device__ __forceinline__ float gauss_of(float u1, float u2)
{
#pragma clang fp contract(off)
    return __builtin_amdgcn_exp2f(-fmaf(u1, u1, u2 * u2));
}

__device__ __forceinline__ float eval_gauss(const float4 &W, float2 c, float lx, float ly)
{
#pragma clang fp contract(off)
    const float u1 = fmaf(ly, W.y, fmaf(lx, W.x, c.x));
    const float u2 = fmaf(ly, W.w, fmaf(lx, W.z, c.y));
    return gauss_of(u1, u2);
}

// alpha of an interpolated splat from a_n, 1 - a_p, 1 - t, t and 1/K; q = (1 -
// a_p)^(1/K).  With t = 0 it is a_n exactly (q is finite).
__device__ __forceinline__ float eval_interp(float an, float omap, float omt, float t, float invK, float &q)
{
#pragma clang fp contract(off)
    q = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(omap) * invK);
    return omt * an + t * (1.0f - q);
}

// True when no pixel of a square of (E + 1) x (E + 1) pixels can take the
// splat at alpha >= 1/255, so that the square may skip it.  On the conic's
// scaled eigen-axes the square's pixel centres lie in the box
// c + [0,E] a + [0,E] b (a = (w1x, w2x), b = (w1y, w2y), c = the offsets of
// its corner pixel), and alpha <= Amax G with G = 2^-(u1^2 + u2^2)
// (Amax = A_n, or max(A_n, A_p) when t > 0: the pow of Eq. (alphap) never
// exceeds its argument).  The distance of the box from the origin is
// compared with log2(255 Amax) with a margin far above the FP32 rounding of
// either side; boxes wider than 64 (sub-pixel splats, whose offsets may
// cancel) are never skipped.
template <int E>
__device__ __forceinline__ bool square_dead(const float4 &W, float c1, float c2, float Amax)
{
    constexpr float e = (float)E;
    const float a1 = e * W.x, b1 = e * W.y, a2 = e * W.z, b2 = e * W.w;
    const float lo1 = c1 + fminf(a1, 0.0f) + fminf(b1, 0.0f), hi1 = c1 + fmaxf(a1, 0.0f) + fmaxf(b1, 0.0f);
    const float lo2 = c2 + fminf(a2, 0.0f) + fminf(b2, 0.0f), hi2 = c2 + fmaxf(a2, 0.0f) + fmaxf(b2, 0.0f);
    if (!(hi1 - lo1 <= 64.0f && hi2 - lo2 <= 64.0f)) return false;
    const float m1 = fmaxf(fmaxf(lo1, -hi1), 0.0f), m2 = fmaxf(fmaxf(lo2, -hi2), 0.0f);
    const float r2 = __builtin_amdgcn_logf(255.0f * Amax);  // log2
    return m1 * m1 + m2 * m2 > r2 * 1.001f + 1e-3f;
}

// Pixel of lane l inside its wave's 8x8 block: quarter l >> 4 is the 4x4
// square at ((q & 1) 4, (q >> 1) 4), rows of four lanes inside it.
__device__ __forceinline__ int quarter_x(int lane) { return ((lane >> 4) & 1) * 4 + (lane & 3); }
__device__ __forceinline__ int quarter_y(int lane) { return (lane >> 5) * 4 + ((lane >> 2) & 3); }

// Quarter mask of a staged splat: bit 4 bk + q set when some pixel of
// quarter q of block bk may take the splat (square_dead on the quarter).
template <int NB>
__device__ __forceinline__ uint32_t quarter_live(const float4 &W, const float2 (&u)[8], float amax)
{
    uint32_t live = 0u;
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float sx = (float)((q & 1) * 4), sy = (float)((q >> 1) * 4);
            const float c1 = fmaf(sy, W.y, fmaf(sx, W.x, u[bk].x)), c2 = fmaf(sy, W.w, fmaf(sx, W.z, u[bk].y));
            live |= square_dead<3>(W, c1, c2, amax) ? 0u : 1u << (4 * bk + q);
        }
    return live;
}

__device__ __forceinline__ int view_of_tile(const DevView *views, int nv, uint32_t tile)
{
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_base <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A splat staged for one tile by the forward.
template <int NB>
struct __align__(16) FwdStaged {
    float4 w;      // axes
    float4 o;      // A_n, A_p, t, 1/K
    float4 c;      // colour, 1 - t
    float2 u[NB];  // per 8x8 block: the offsets of its corner pixel on the axes
    static constexpr uint32_t kStride = 16u * ((uint32_t)(3 + (NB + 1) / 2) | 1u);  // odd units: banks apart
};

// Whether the quarters of the block may take the staged splat: bit 4 bk + q.
template <int NB, int SX>
__device__ __forceinline__ uint32_t stage_fwd(const SplatRec &r, const double4 &W64, int ox, int oy,
                                              FwdStaged<NB> &st)
{
    const float4 W = make_float4((float)W64.x, (float)W64.y, (float)W64.z, (float)W64.w);
    float2 u[8];
    st.w = W;
    st.o = make_float4(r.An, r.Ap, r.t, r.invK);
    st.c = make_float4(r.r, r.g, r.b, 1.0f - r.t);
#pragma unroll
    for (int bk = 0; bk < NB; ++bk) {
        float c1, c2, d0, d1;
        block_offsets(r, W64, ox + (bk % SX) * 8, oy + (bk / SX) * 8, c1, c2, d0, d1);
        st.u[bk] = u[bk] = make_float2(c1, c2);
    }
    return quarter_live<NB>(W, u, r.t > 0.0f ? fmaxf(r.An, r.Ap) : r.An);
}

// Per-wave work counts (uint4 per wave, plain stores) are summed by
// k_stats_reduce into three consecutive counters: forward (evaluated,
// blended, evaluated with t > 0), backward (evaluated, evaluated with t > 0,
// contributing).  No contended atomics on the hot path.

// Work distribution over tiles: either one workgroup per tile slot (grid =
// tile count, slot = workgroup index), or a persistent grid sized to the
// chip's resident workgroups, each taking runs of `chunk` consecutive slots
// from a device-side queue (a counter that the launch sequence clears first)
// until the slots run out.  Slots are handed out in the longest-first order
// either way; runs keep the one queue counter from serialising a million
// small tiles.
__device__ __forceinline__ uint32_t next_run(uint32_t *queue, uint32_t chunk, uint32_t *s_slot)
{
    if (threadIdx.x == 0) *s_slot = atomicAdd(queue, chunk);
    __syncthreads();
    const uint32_t slot = *s_slot;
    __syncthreads();  // every wave has its slot before lane 0 may overwrite it
    return slot;
}

// OR over each row of 16 lanes (DPP partners l ^ 8, l ^ 7, l ^ 2, l ^ 1).
__device__ __forceinline__ uint32_t row_or(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
    return v;
}

// The forward of one tile.  Bound by VALU issue where many tiles are resident,
// by the latency of one step where few are (a tile's pixels walk up to
// thousands of splats in turn).  A quarter walks a list of the entries it may
// take, made per chunk of 128 staged entries, two entries at a time: the two
// alphas are independent, and the list costs one read where taking apart a
// bit mask cost seven instructions a step.
//
// An FP32 multiply, add or FMA on vector registers issues in 2 cycles here (2.2
// measured), with a scalar register among its operands in 4 (4.1), as a compare,
// select, minimum or lane exchange (4.2), exp2 and log2 in 8 (8.1): what a step
// keeps per pixel is therefore its colour, its transmittance and one
// history bit (an add with carry), from which count and last contributor
// follow every 32 entries, and which lanes still run is a scalar mask.  45
// instructions a step in place of 61.  32 views of 1920x1080 over 30M leaves:
// 16x8 tiles 5.1 -> 4.3 ms, 8x8 4.4 -> 4.1, 16x16 6.6 -> 4.7, 32x16 14.2 ->
// 7.4; one view with 16x16 tiles 561 -> 460 us, of 1M leaves 288 -> 236 us.
// (Records read by one ds_read_b32 a lane and taken from each other's
// registers by row_newbcast leave the LDS nearly idle but cost a 4-cycle move
// for every operand of an FMA: 5.4 ms.)
template <int TW, int TH>
__device__ __forceinline__ void blend_tile(const DevView *__restrict__ views, int nv,
                                           const uint32_t *__restrict__ tile_order,
                                           const uint2 *__restrict__ ranges, const uint32_t *__restrict__ pair_vals,
                                           const SplatRec *__restrict__ recs, const double4 *__restrict__ axes,
                                           float *__restrict__ T_final, uint32_t *__restrict__ n_last,
                                           uint32_t *__restrict__ n_blend, uint8_t *__restrict__ qbits,
                                           uint32_t qstride, uint4 *__restrict__ wstats, uint32_t slot)
{
    constexpr int NT = TW * TH;
    constexpr int NW = NT / 64;
    constexpr int SX = TW / 8;
    constexpr int NB = (TW / 8) * (TH / 8);
    constexpr int BATCH = NT;  // records staged at a time: one per thread
    constexpr int CH = BATCH < 128 ? BATCH : 128;  // entries per list
    constexpr int LIST = CH + 4;
    static_assert(BATCH % CH == 0 && CH % 64 == 0 && NB <= 8, "tile");
    using Rec = FwdStaged<NB>;
    constexpr uint32_t kRec = Rec::kStride, kDead = kRec * BATCH;
    static_assert(sizeof(Rec) <= kRec && kDead < 65536, "a list entry is a 16-bit byte offset");
    // the last record has alpha 0 everywhere: for a quarter past its list's end
    __shared__ __align__(16) unsigned char s_rec[kRec * (BATCH + 1)];
    __shared__ uint32_t s_qm[NB][4][BATCH / 32];  // bit b of word k: quarter q of block bk may take entry 32 k + b
    __shared__ __align__(4) uint16_t s_list[NB][4][LIST];  // the records a quarter walks (byte offsets in s_rec)
    __shared__ uint32_t s_hit[NB][4][CH / 32];  // of the chunk: the entries some pixel of the quarter blended
    const uint32_t tile = tile_order[slot];  // longest lists first
    const int vi = view_of_tile(views, nv, tile);
    const DevView &V = views[vi];
    const uint32_t lt = tile - V.tile_base;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4, ql = lane & 15;
    const int ox = tx * TW, oy = ty * TH;
    const int bx = quarter_x(lane), by = quarter_y(lane);
    const int px = ox + (w % SX) * 8 + bx, py = oy + (w / SX) * 8 + by;
    const bool inside = px < V.W && py < V.H;
    const float lx = (float)bx, ly = (float)by;
    const uint2 rg = ranges[tile];
    // alive: the lanes whose pixel is inside the image and not finished.  A
    // pixel stops at the splat whose blend would take T below kTMin; that
    // splat was evaluated but not blended.
    uint64_t alive = __builtin_amdgcn_ballot_w64(inside);
    float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
    uint32_t last = 0, nb = 0;
    uint32_t n_eval = 0, n_eval_t = 0;  // wave totals (scalar): evaluated pairs, of them interpolated

    // index of this thread's record of the next batch, loaded while the current
    // one is composited (loading the records ahead too took 20 registers a lane:
    // with two waves fewer per SIMD the headline batch of 32 views lost 0.7 ms)
    uint32_t nxt = 0;
    auto fetch = [&](uint32_t b0) {
        if (b0 + threadIdx.x < rg.y) nxt = pair_vals[b0 + threadIdx.x];
    };
    if (rg.x < rg.y) fetch(rg.x);
    if (threadIdx.x < kRec / 4)  // (ordered before its first read by the barriers below)
        reinterpret_cast<float *>(s_rec + kDead)[threadIdx.x] = 0.0f;
    for (uint32_t b0 = rg.x; b0 < rg.y; b0 += BATCH) {
        if (!__syncthreads_or(alive != 0ull)) break;
        {
            uint32_t live = 0u;
            if (b0 + threadIdx.x < rg.y)
                live = stage_fwd<NB, SX>(recs[nxt], axes[nxt], ox, oy,
                                         *reinterpret_cast<Rec *>(s_rec + kRec * threadIdx.x));
#pragma unroll
            for (int bq = 0; bq < 4 * NB; ++bq) {
                const uint64_t m = __ballot((live >> bq) & 1u);
                if (lane < 2) s_qm[bq >> 2][bq & 3][2 * w + lane] = (uint32_t)(lane ? m >> 32 : m);
            }
        }
        __syncthreads();
        if (b0 + BATCH < rg.y) fetch(b0 + BATCH);
        const int cnt = (int)min((uint32_t)BATCH, rg.y - b0);
        for (int c0 = 0; c0 < cnt && alive != 0ull; c0 += CH) {
            // the entries of the chunk that each unfinished quarter may take, in
            // order; two quarters at a time, one lane per entry
            const int n_ch = min(cnt - c0, CH);
            if (lane < 4 * (CH / 32)) (&s_hit[w][0][0])[lane] = 0u;
            for (int k = 0; k < n_ch + 4; k += 32)
                if (k + 2 * ql < LIST) reinterpret_cast<two_u16 *>(&s_list[w][q][0])[k / 2 + ql] = kDead * 0x10001u;
            int steps = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int qa = 2 * h + (lane >> 5), i = lane & 31;
                const bool open = ((alive >> (16 * qa)) & 0xFFFFull) != 0ull;
                int n = 0;
#pragma unroll
                for (int k = 0; k < CH / 32; ++k) {
                    if (32 * k >= n_ch) break;
                    const uint32_t m = open ? s_qm[w][qa][c0 / 32 + k] : 0u;
                    if ((m >> i) & 1u)
                        s_list[w][qa][n + __popc(m & ((1u << i) - 1u))] = (uint16_t)((c0 + 32 * k + i) * kRec);
                    n += __popc(m);
                }
                steps = max(steps, max(__builtin_amdgcn_readlane(n, 0), __builtin_amdgcn_readlane(n, 32)));
            }
            steps = __builtin_amdgcn_readfirstlane(steps);
            wave_lds_sync();  // the lists are this wave's own
            const uint16_t *list = &s_list[w][q][0];
            const two_u16 *walk = reinterpret_cast<const two_u16 *>(list);
            // history: the pixel blended (or stopped at) the entry, the latest
            // entry in bit 0; alive0: alive when it was last emptied
            uint32_t hist = 0u;
            uint64_t alive0 = alive;
            // the history's m list entries from position p0 into count, last
            // contributor and the quarters' hits
            auto flush = [&](int p0, int m) {
                const bool died = __builtin_amdgcn_inverse_ballot_w64(alive0 & ~alive);
                const uint32_t blended = died ? hist & (hist - 1u) : hist;  // not the splat a pixel stopped at
                nb += (uint32_t)__popc(blended);
                if (blended)  // 1-based list position
                    last = b0 - rg.x + (uint32_t)list[p0 + m - 1 - __builtin_ctz(blended)] / kRec + 1u;
                const uint32_t hits = row_or(hist);
                hist = 0u;
                alive0 = alive;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int bit = 16 * h + ql;
                    if ((hits >> bit) & 1u) {
                        const uint32_t e = (uint32_t)list[p0 + m - 1 - bit] / kRec - (uint32_t)c0;
                        atomicOr(&s_hit[w][q][e >> 5], 1u << (e & 31u));
                    }
                }
            };
            uint32_t two = walk[0];
            int p = 0;
            while (p < steps) {
                const uint32_t off[2] = {two & 0xFFFFu, two >> 16};
                const uint64_t h0 = __builtin_amdgcn_ballot_w64(off[0] < kDead);
                if ((alive & h0) == 0ull) break;  // every quarter is finished or past its list's end
                two = walk[(p >> 1) + 1];
                const uint64_t hm[2] = {h0, __builtin_amdgcn_ballot_w64(off[1] < kDead)};
                float4 Ov[2], Cc[2];
                float G[2], al[2];
                uint64_t tm[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const Rec &r = *reinterpret_cast<const Rec *>(s_rec + off[s]);
                    const float4 Wv = r.w;
                    Ov[s] = r.o;
                    Cc[s] = r.c;
                    G[s] = eval_gauss(Wv, r.u[w], lx, ly);
                    al[s] = fminf(Ov[s].x * G[s], kAlphaMax);
                    tm[s] = __builtin_amdgcn_ballot_w64(Ov[s].z > 0.0f);
                }
                if (tm[0] | tm[1]) {  // with t = 0 the interpolated form gives a_n exactly
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        float qp;
                        al[s] = eval_interp(al[s], 1.0f - fminf(Ov[s].y * G[s], kAlphaMax), Cc[s].w, Ov[s].z, Ov[s].w,
                                            qp);
                    }
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    // masks and work counts on the scalar unit
                    const uint64_t gm = hm[s] & alive;
                    n_eval += (uint32_t)__popcll(gm);
                    n_eval_t += (uint32_t)__popcll(gm & tm[s]);
                    const uint64_t go = alive & __builtin_amdgcn_ballot_w64(al[s] >= kAlphaMin);
                    const float Tn = T * (1.0f - al[s]);
                    const uint64_t on = go & ~__builtin_amdgcn_ballot_w64(Tn < kTMin);
                    const bool lon = __builtin_amdgcn_inverse_ballot_w64(on);
                    const float wgt = lon ? al[s] * T : 0.0f;
                    C0 = fmaf(Cc[s].x, wgt, C0);
                    C1 = fmaf(Cc[s].y, wgt, C1);
                    C2 = fmaf(Cc[s].z, wgt, C2);
                    T = lon ? Tn : T;
                    // the splat a pixel stops at too: the backward drops it
                    hist = hist + hist + (__builtin_amdgcn_inverse_ballot_w64(go) ? 1u : 0u);
                    alive &= ~(go ^ on);
                }
                p += 2;
                if ((p & 31) == 0) flush(p - 32, 32);
            }
            if (p & 31) flush(p & ~31, p & 31);
            wave_lds_sync();
            // the backward takes, per quarter, only the entries it blended here
            // (entries after the last chunk walked lie after every pixel's last
            // contributor, where the backward never looks): the byte of every
            // entry of the chunk, bit q for quarter q, into the block's plane
            for (int k = 0; k < n_ch; k += 64) {
                const int e = k + lane;
                uint32_t byte = 0u;
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) byte |= ((s_hit[w][qq][e >> 5] >> (e & 31)) & 1u) << qq;
                if (e < n_ch) qbits[(size_t)w * qstride + b0 + (uint32_t)(c0 + e)] = (uint8_t)byte;
            }
            wave_lds_sync();  // read before the next chunk clears it
        }
    }
    if (inside) {
        const size_t p = (size_t)py * V.W + px;
        float *o = V.out_rgb + 3 * p;
        o[0] = C0;
        o[1] = C1;
        o[2] = C2;
        const size_t g = (size_t)V.pix_base + p;
        T_final[g] = T;
        n_last[g] = last;
        n_blend[g] = nb;
    }
    uint32_t nb_w = nb;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) nb_w += (uint32_t)__shfl_xor((int)nb_w, d, 64);
    if (lane == 0) wstats[(size_t)slot * NW + w] = make_uint4(n_eval, nb_w, n_eval_t, 0u);
}

template <int TW, int TH, bool PERSIST>
__global__ __launch_bounds__(TW *TH) void k_blend(const DevView *__restrict__ views, int nv,
                                                  const uint32_t *__restrict__ tile_order,
                                                  const uint2 *__restrict__ ranges,
                                                  const uint32_t *__restrict__ pair_vals,
                                                  const SplatRec *__restrict__ recs,
                                                  const double4 *__restrict__ axes, float *__restrict__ T_final,
                                                  uint32_t *__restrict__ n_last, uint32_t *__restrict__ n_blend,
                                                  uint8_t *__restrict__ qbits, uint32_t qstride,
                                                  uint4 *__restrict__ wstats, uint32_t n_tiles,
                                                  uint32_t *__restrict__ queue, uint32_t chunk)
{
    if constexpr (!PERSIST) {
        blend_tile<TW, TH>(views, nv, tile_order, ranges, pair_vals, recs, axes, T_final, n_last, n_blend,
                                  qbits, qstride, wstats, blockIdx.x);
    } else {
        __shared__ uint32_t s_slot;
        for (;;) {
            const uint32_t first = next_run(queue, chunk, &s_slot);
            if (first >= n_tiles) break;
            const uint32_t last = min(n_tiles, first + chunk);
            for (uint32_t slot = first; slot < last; ++slot) {
                blend_tile<TW, TH>(views, nv, tile_order, ranges, pair_vals, recs, axes, T_final, n_last,
                                          n_blend, qbits, qstride, wstats, slot);
                __syncthreads();  // LDS of this tile read by every wave before the next stages
            }
        }
    }
}

// Sums over each row of 16 lanes (one 4x4 quarter of the wave's block) of 12
// per-lane values, taken as six pairs: four halvings with DPP inside the row
// (partners l ^ 8, l ^ 7, l ^ 2 and l ^ 1), each keeping one of the two
// values of a pair per lane.  A: the pairs after the first halving.  Lane l of
// the row ends with the row's total of value row_slot(l) (value 2 k + 1 is the
// second of pair k; -1: a copy of another lane's total).
//
// In the second halving the lanes that keep a pair's first value are whole
// banks of 4 (lanes l with l & 4 clear): two adds under bank masks instead of
// two selects and an add.  Every lane must be active.  (The leading s_nop
// covers the two wait states that a DPP operand needs after the VALU wrote
// it.)
__device__ __forceinline__ void halve_l7(const float (&A)[6], float (&B)[3])
{
#define HGS_HALF(o, f, s)                                                                                  \
    "v_add_f32_dpp " o ", " f ", " f " row_half_mirror row_mask:0xf bank_mask:0x5\n\t"                    \
    "v_add_f32_dpp " o ", " s ", " s " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
    asm("s_nop 1\n\t" HGS_HALF("%0", "%3", "%4") HGS_HALF("%1", "%5", "%6") HGS_HALF("%2", "%7", "%8")
        : "=&v"(B[0]), "=&v"(B[1]), "=&v"(B[2])
        : "v"(A[0]), "v"(A[1]), "v"(A[2]), "v"(A[3]), "v"(A[4]), "v"(A[5]));
#undef HGS_HALF
}
// The first halving of a pair without products (banks 0 and 1 keep the first).
__device__ __forceinline__ float halve_l8(float first, float second)
{
    float o;
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        : "=&v"(o)
        : "v"(first), "v"(second));
    return o;
}

__device__ __forceinline__ float row_reduce12(const float (&A)[6], int lane)
{
    const bool b1 = (lane & 2) != 0, b0 = (lane & 1) != 0;
    float B[3];
    halve_l7(A, B);
    const float C0 = (b1 ? B[1] : B[0]) + dpp_move<0x4E>(b1 ? B[0] : B[1]);
    const float C1 = B[2] + dpp_move<0x4E>(B[2]);
    return (b0 ? C1 : C0) + dpp_move<0xB1>(b0 ? C0 : C1);
}

__device__ __forceinline__ int row_slot(int lane)
{
    const int b3 = (lane >> 3) & 1, b2 = (lane >> 2) & 1, b1 = (lane >> 1) & 1, b0 = lane & 1;
    return b0 == 0 ? 4 * b1 + 2 * b2 + b3 : (b1 == 0 ? 8 + 2 * b2 + b3 : -1);
}

constexpr int kG = 12;  // floats per splat in the screen-space gradient

// Gradient slots of a splat, summed over the pixels of the tile.  With h = G
// dL/dG (G the Gaussian) and (x, y) the pixel's offset from the tile centre:
//   0, 1    h x, h y
//   2, 3    h x x, h y y
//   4       h x y
//   5       S = h
//   6, 7    dL/dA_n, dL/dA_p (A = kappa |o|)
//   8..10   dL/d colour
//   11      dL/dt through alpha (only when the caller asks for dL/dt)
// The flush maps the moments by the conic's scaled eigen-axes (v = W (x, y),
// u = v + c, c the tile centre's offset formed in FP64 at staging) and about
// the splat's centre, in FP64: P = P' + c S and Q = Q' + c P'^T + P' c^T +
// c c^T S.  Taken directly about the splat's centre, the moments of a large
// splat whose centre lies far off screen are dominated by c S and c c^T S,
// and the mean and covariance gradients built from them cancel almost
// entirely in the chain through the projection: separately rounded FP32 sums
// of P and Q then leave errors far above the result.  With the moments about
// the tile both large parts carry the one rounded S, and the cancellation
// removes its error with it.  What remains is the FP32 rounding of the
// moments, which grows with the squared offset: hence the tile's centre
// (at most half the tile's diagonal) rather than a corner, and S summed from
// the same per-pixel h (forming it from slots 6 and 7 instead, equal in exact
// arithmetic, leaves per-pixel differences that c c^T amplifies).
// The screen-space gradient follows from the tile sums by the splat's
// (per-tile constant) axes: with g = conic d = (u1 w1 + u2 w2) / kHalfLog2e
// and G = exp(-q/2), dL/dmean = sum h g and dL/dSigma2' = -sum (h / 2) g g^T
// (the covariance gradient through the conic), both linear in P and Q.
__device__ __forceinline__ void screen_grad(const float4 &W, const double P[2], const double Q[3], double out[5])
{
    const double k = 1.0 / kHalfLog2e;
    const double wx = W.x, wy = W.y, wz = W.z, ww = W.w;
    const double P1 = P[0], P2 = P[1], Q11 = Q[0], Q12 = Q[1], Q22 = Q[2];
    out[0] = k * (wx * P1 + wz * P2);
    out[1] = k * (wy * P1 + ww * P2);
    // (a, b, c) = (xx, 2 xy, yy) of sum (h / 2) g g^T, entering dL/dSigma2' with a minus
    // sign that the chain below takes as -dq = h / 2
    out[2] = 0.5 * k * k * (wx * wx * Q11 + 2.0 * wx * wz * Q12 + wz * wz * Q22);
    out[3] = k * k * (wx * wy * Q11 + (wx * ww + wz * wy) * Q12 + wz * ww * Q22);
    out[4] = 0.5 * k * k * (wy * wy * Q11 + 2.0 * wy * ww * Q12 + ww * ww * Q22);
}

// Offsets of the centre of the TW x TH tile at (ox, oy) on the scaled
// eigen-axes, in FP64.
template <int TW, int TH>
__device__ __forceinline__ double2 centre_offsets(const SplatRec &r, const double4 &W, int ox, int oy)
{
#pragma clang fp contract(off)
    const double dx = ((double)(ox - r.ax) + 0.5 * TW) - (double)r.fx;
    const double dy = ((double)(oy - r.ay) + 0.5 * TH) - (double)r.fy;
    return make_double2(dx * W.x + dy * W.y, dx * W.z + dy * W.w);
}

// Reduction.  Each step (one splat per quarter, one pixel per lane) leaves 12
// values per lane: the moments of h about the tile's centre on the splat's
// axes, dL/dA_n, dL/dA_p, the colours and dL/dt.  They are summed over the
// quarter's row of 16 lanes by four DPP halvings, and the totals go to the
// tile's LDS sums (FP64 atomics).
//
// The order of the operations is written out, every FMA: large splats near the
// eye cancel almost all of their moments, and any other form or order moves
// single elements of the scale and rotation gradients (sums over a column
// first and pixel moments at the flush: by up to 2e-3 of their RMS on 32x16
// tiles, 5e-4 on smaller ones).  An L1 cotangent of a second step then differs
// in sign where image and target meet, so that results would change from one
// version to the next far beyond rounding.  That form took 7.4 ms where this
// one takes 7.9 (32 views of 1920x1080 over 30M leaves, 16x8 tiles).
//
// The kernel issues VALU instructions near the limit, so what counts is their
// number per step: the walk's order is a list made per batch instead of a bit
// mask taken apart step by step, two entries are taken at a time, and a record
// sits at one LDS address.  v_mfma_f32_16x16x4_f32 for the sums was slower
// (FP32 matrix instructions hold the VALU for their 32 cycles: 11.5 against
// 9.0 ms), larger batches too (7.6 -> 8.9 ms at 128 entries: fewer tiles
// resident).  Of the last steps, the halvings under bank masks gave 8.4 ->
// 8.1 ms and the cotangent's selects kept in registers 8.1 -> 7.9.  From one
// entry a step found in a bit mask: 9.2 -> 7.9 ms; 16x16 tiles 10.0 -> 7.7,
// 32x16 19.2 -> 9.7; 8 views of 1280x720 over 2M leaves
// 4.2 -> 3.5 ms.
//
// DET (the deterministic mode): no floating-point atomics.  Each quarter
// stores its FP32 partial sums in a slot of its own, the flush adds the
// quarters in a fixed order (FP64), and the tile's 11 terms for a splat go
// with plain stores to det.part at the pair's position in the list
// k_duplicate emitted (the splat's first pair plus the tile's row-major index
// in its tile rectangle); launch_det_sum then adds each splat's rows in order.

// A splat staged for one tile by the backward.
template <int NB>
struct __align__(16) BwdStaged {
    float4 w;      // axes
    float4 o;      // A_n, A_p, t, 1/K
    float4 c;      // colour, 1 - t
    float2 u[NB];  // per 8x8 block: the offsets of its corner pixel on the axes
    double g[kG];  // the tile's sums; the flush turns them into the splat's 11 terms in place
    // Bytes from one record to the next: an odd number of 16-byte units, so
    // that the different records that the four quarters of a wave read at once
    // collide in a bank for a distance of 16 records only (LDS conflict
    // cycles of the 8 x 1280x720 workload 0.21 -> 0.11 of the kernel's time).
    static constexpr uint32_t kStride = 16u * ((uint32_t)(3 + (NB + 1) / 2 + kG / 2) | 1u);
};

template <int TW, int TH, bool DT, bool DET>
__device__ __forceinline__ void blend_bwd_tile(const DevView *__restrict__ views, int nv,
                                               const uint32_t *__restrict__ tile_order,
                                               const uint2 *__restrict__ ranges,
                                               const uint32_t *__restrict__ pair_vals,
                                               const SplatRec *__restrict__ recs, const double4 *__restrict__ axes,
                                               const float *__restrict__ T_final,
                                               const uint32_t *__restrict__ n_last,
                                               const uint8_t *__restrict__ qbits, uint32_t qstride,
                                               const uint32_t *__restrict__ vis_rank, double *__restrict__ sgrad,
                                               const DetArgs det, uint4 *__restrict__ wstats, uint32_t tslot)
{
    constexpr int NT = TW * TH;
    constexpr int NW = NT / 64;
    constexpr int SX = TW / 8;
    constexpr int NB = (TW / 8) * (TH / 8);
    constexpr int PER = 32;  // entries that a wave stages and flushes
    constexpr int BATCH = DET ? PER : PER * NW;
    constexpr int NQW = BATCH / 32;  // 32-entry words of a quarter's mask
    static_assert(NB <= 8, "tile");
    using Rec = BwdStaged<NB>;
    constexpr uint32_t kRec = Rec::kStride, kDead = kRec * BATCH;
    static_assert(sizeof(Rec) <= kRec && kDead < 65536, "a list entry is a 16-bit byte offset");
    // the last record blends nowhere: for a quarter past its list's end
    __shared__ __align__(16) unsigned char s_rec[kRec * (BATCH + 1)];
    auto rec_at = [&](uint32_t off) -> Rec & { return *reinterpret_cast<Rec *>(s_rec + off); };
    __shared__ uint32_t s_id[BATCH];  // gradient rows
    __shared__ float s_gr[DET ? 4 * NW : 1][DET ? BATCH : 1][kG];  // DET: each quarter's partial sums
    __shared__ uint32_t s_pq[DET ? BATCH : 1];  // DET: the pair's position in the emitted list
    __shared__ double2 s_ref[BATCH];    // the tile centre's offsets on the axes (FP64)
    __shared__ uint32_t s_qm[NB][4][NQW];     // bit b of word k: quarter q of block bk blended entry 32 k + b
    // the records a quarter walks, back to front (byte offsets in s_r)
    constexpr int LIST = BATCH + 4;
    __shared__ __align__(4) uint16_t s_list[NB][4][LIST];
    __shared__ uint32_t s_max;
    const uint32_t tile = tile_order[tslot];  // longest lists first
    const int vi = view_of_tile(views, nv, tile);
    const DevView &V = views[vi];
    const uint32_t lt = tile - V.tile_base;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4;
    const int ox = tx * TW, oy = ty * TH;
    const int bx = quarter_x(lane), by = quarter_y(lane);
    const int px = ox + (w % SX) * 8 + bx, py = oy + (w / SX) * 8 + by;
    const bool inside = px < V.W && py < V.H;
    const float lx = (float)bx, ly = (float)by;
    const uint2 rg = ranges[tile];

    // the pixel's offset from the tile centre, this lane's slot, and
    // which value of each pair it keeps in the first halving
    const float lxt = (float)(px - ox) - 0.5f * (TW - 1), lyt = (float)(py - oy) - 0.5f * (TH - 1);
    const int slot = row_slot(lane);
    const bool b3 = (lane & 8) != 0;

    float T = 1.0f, g0 = 0.0f, g1 = 0.0f, g2 = 0.0f;
    uint32_t last = 0;
    if (inside) {
        const size_t p = (size_t)py * V.W + px;
        const size_t g = (size_t)V.pix_base + p;
        T = T_final[g];
        last = n_last[g];
        g0 = V.dL[3 * p];
        g1 = V.dL[3 * p + 1];
        g2 = V.dL[3 * p + 2];
    }
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    // the cotangent as the first halving takes it (pairs (0, 1) and (2, -)),
    // kept in registers: the compiler would select anew in every step
    float ga = b3 ? g1 : g0, gb = b3 ? g0 : g1, g2a = b3 ? 0.0f : g2, g2b = b3 ? g2 : 0.0f;
    asm volatile("" : "+v"(ga), "+v"(gb), "+v"(g2a), "+v"(g2b));
    // the quarter's last contributor, then the tile's
    uint32_t qm = last;
    qm = max(qm, (uint32_t)__shfl_xor((int)qm, 1, 64));
    qm = max(qm, (uint32_t)__shfl_xor((int)qm, 2, 64));
    qm = max(qm, (uint32_t)__shfl_xor((int)qm, 4, 64));
    qm = max(qm, (uint32_t)__shfl_xor((int)qm, 8, 64));
    uint32_t wm = max(qm, (uint32_t)__shfl_xor((int)qm, 16, 64));
    wm = max(wm, (uint32_t)__shfl_xor((int)wm, 32, 64));
    if (lane == 0) atomicMax(&s_max, wm);
    __syncthreads();
    const uint32_t end = rg.x + s_max;
    float R0 = 0.0f, R1 = 0.0f, R2 = 0.0f;  // colour composited behind the current splat
    uint32_t n_eval = 0, n_eval_t = 0, n_con = 0;  // wave totals (scalar)

    if (threadIdx.x == 0) {  // (ordered before its first read by the barrier after the staging)
        Rec &dead = rec_at(kDead);
        dead.w = dead.o = dead.c = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int bk = 0; bk < NB; ++bk) dead.u[bk] = make_float2(0.0f, 0.0f);
    }

    for (uint32_t hi = end; hi > rg.x;) {
        const uint32_t lo = hi - rg.x > (uint32_t)BATCH ? hi - BATCH : rg.x;
        const int cnt = (int)(hi - lo);
        {
            // wave w stages entries PER w .. PER w + PER - 1, so that the
            // staging work is spread over the waves of the tile
            const int j = PER * w + lane;
            uint32_t live = 0u;
            if (lane < PER && j < cnt) {
                const uint32_t sidx = pair_vals[lo + j];
                const SplatRec r = recs[sidx];
                const double4 W64 = axes[sidx];
                const float4 W = make_float4((float)W64.x, (float)W64.y, (float)W64.z, (float)W64.w);
                Rec &sr = rec_at(kRec * (uint32_t)j);
#pragma unroll
                for (int bk = 0; bk < NB; ++bk) {
                    float c1, c2, d0, d1;
                    block_offsets(r, W64, ox + (bk % SX) * 8, oy + (bk / SX) * 8, c1, c2, d0, d1);
                    sr.u[bk] = make_float2(c1, c2);
                    // the quarters of this block that blended the splat in the forward
                    live |= (uint32_t)qbits[(size_t)bk * qstride + lo + (uint32_t)j] << (4 * bk);
                }
                s_id[j] = vis_rank[sidx];
                sr.w = W;
                sr.o = make_float4(r.An, r.Ap, r.t, r.invK);
                auto colour = [](float c) { return signbit(c) ? __builtin_inff() : c; };
                sr.c = make_float4(colour(r.r), colour(r.g), colour(r.b), 1.0f - r.t);
                s_ref[j] = centre_offsets<TW, TH>(r, W64, ox, oy);
                if constexpr (DET) {
                    for (int row = 0; row < 4 * NW; ++row)
#pragma unroll
                        for (int k = 0; k < kG; ++k) s_gr[row][j][k] = 0.0f;
                    const uint32_t jr = det.jrank[sidx];
                    const uint2 rc = det.rect[jr];
                    const uint32_t tx0 = rc.x & 0xFFFFu, tx1 = rc.x >> 16, ty0 = rc.y & 0xFFFFu;
                    s_pq[j] = det.pair_offsets[jr] + ((uint32_t)ty - ty0) * (tx1 - tx0 + 1u) + ((uint32_t)tx - tx0);
                } else {
#pragma unroll
                    for (int k = 0; k < kG; ++k) sr.g[k] = 0.0;
                }
            }
            if (PER * w < BATCH) {  // this wave's words of the quarter masks
#pragma unroll
                for (int bq = 0; bq < 4 * NB; ++bq) {
                    const uint64_t m = __ballot((live >> bq) & 1u);
                    if (lane < PER / 32) s_qm[bq >> 2][bq & 3][PER / 32 * w + lane] = (uint32_t)(lane ? m >> 32 : m);
                }
            }
        }
        __syncthreads();
        // the entries each quarter of this wave's block walks: those some pixel
        // of it blended in the forward, before its last contributor (later
        // records are not written); two quarters at a time, one lane per
        // entry, the rest of the list filled with the dead record
        const uint32_t base = lo - rg.x;  // list position of entry 0
        int steps = 0;                    // entries of the longest list
#pragma unroll
        for (int k = 0; k < 4 * LIST / 2; k += 64)
            if (k + 64 <= 4 * LIST / 2 || k + lane < 4 * LIST / 2)
                reinterpret_cast<two_u16 *>(&s_list[w][0][0])[k + lane] = kDead * 0x10001u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int qa = 2 * h + (lane >> 5), i = lane & 31;
            const uint32_t qma = (uint32_t)__builtin_amdgcn_readlane((int)qm, 32 * h),
                           qmb = (uint32_t)__builtin_amdgcn_readlane((int)qm, 32 * h + 16);
            const uint32_t lastq = lane < 32 ? qma : qmb;
            const int limq = lastq > base ? (int)min(lastq - base, (uint32_t)cnt) : 0;
            int n = 0;
#pragma unroll
            for (int k = NQW - 1; k >= 0; --k) {
                const int lk = limq - 32 * k;  // entries 32 k + i, i < lk, come before the last contributor
                uint32_t m = 32 * k < cnt ? s_qm[w][qa][k] : 0u;
                m &= lk >= 32 ? ~0u : (lk <= 0 ? 0u : (1u << lk) - 1u);
                if ((m >> i) & 1u) s_list[w][qa][n + __popc((m >> i) >> 1)] = (uint16_t)((32 * k + i) * kRec);
                n += __popc(m);
            }
            steps = max(steps, max(__builtin_amdgcn_readlane(n, 0), __builtin_amdgcn_readlane(n, 32)));
        }
        steps = __builtin_amdgcn_readfirstlane(steps);
        wave_lds_sync();  // the lists are this wave's own
        // each quarter walks its list, the four quarters of the wave together,
        // two entries at a time
        const two_u16 *walk = reinterpret_cast<const two_u16 *>(&s_list[w][q][0]);
        const uint32_t lim = (uint32_t)min((int)(last - min(last, base)), cnt) * kRec;  // the pixel's last contributor
        uint32_t two = walk[0];
        for (int p = 0; p < steps; p += 2) {
            const uint32_t off[2] = {two & 0xFFFFu, two >> 16};
            two = walk[(p >> 1) + 1];
            float4 Ov[2], Wv[2], Cv[2];
            float G[2], al[2], anr[2], apr[2], omt[2], omap[2], qp[2];
            bool con[2];
            uint64_t tm[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const Rec &r = rec_at(off[s]);
                Cv[s] = r.c;
                Wv[s] = r.w;
                Ov[s] = r.o;
                omt[s] = Cv[s].w;
                tm[s] = __builtin_amdgcn_ballot_w64(Ov[s].z > 0.0f);
                G[s] = eval_gauss(Wv[s], r.u[w], lx, ly);
                anr[s] = Ov[s].x * G[s];
                al[s] = fminf(anr[s], kAlphaMax);
                apr[s] = 0.0f;
                omap[s] = qp[s] = 1.0f;
            }
            const bool any_t = (tm[0] | tm[1]) != 0ull;  // with t = 0 the interpolated form gives a_n exactly
            if (any_t) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    apr[s] = Ov[s].y * G[s];
                    omap[s] = 1.0f - fminf(apr[s], kAlphaMax);
                    al[s] = eval_interp(al[s], omap[s], omt[s], Ov[s].z, Ov[s].w, qp[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                // lane masks straight from the compares
                const uint64_t irm = __builtin_amdgcn_ballot_w64(off[s] < lim);
                n_eval += (uint32_t)__popcll(irm);
                n_eval_t += (uint32_t)__popcll(irm & tm[s]);
                n_con += (uint32_t)__popcll(irm & __builtin_amdgcn_ballot_w64(al[s] >= kAlphaMin));
                con[s] = off[s] < lim && al[s] >= kAlphaMin;
            }
            float dan[2], dap[2], aT[2], dal[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                // under the lane mask: with a = 0 for the others an infinite colour
                // would make NaN of their R
                dal[s] = aT[s] = 0.0f;
                if (con[s]) {
                    const float a = al[s];
                    T = T * __builtin_amdgcn_rcpf(1.0f - a);
                    aT[s] = a * T;
                    const float d0 = Cv[s].x - R0, d1 = Cv[s].y - R1, d2 = Cv[s].z - R2;
                    dal[s] = T * fmaf(d2, g2, fmaf(d0, g0, d1 * g1));
                    R0 = fmaf(a, d0, R0);
                    R1 = fmaf(a, d1, R1);
                    R2 = fmaf(a, d2, R2);
                }
            }
            // dL/da_n, dL/da_p (zero through the clamps)
            if (any_t) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    // d alpha' / d a_p = (1/K) (1 - a_p)^(1/K - 1) = (1/K) q / (1 - a_p)
                    const float dp = (Ov[s].z * dal[s]) * Ov[s].w * (qp[s] * __builtin_amdgcn_rcpf(omap[s]));
                    dan[s] = con[s] && !(anr[s] > kAlphaMax) ? omt[s] * dal[s] : 0.0f;
                    dap[s] = con[s] && !(apr[s] > kAlphaMax) ? dp : 0.0f;
                }
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    dan[s] = con[s] && !(anr[s] > kAlphaMax) ? dal[s] : 0.0f;
                    dap[s] = 0.0f;
                }
            }
            float dt[2] = {0.0f, 0.0f};  // dL/dt through alpha: (a'_p - a_n) dL/dalpha
            if constexpr (DT)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    dt[s] = con[s] && Ov[s].z > 0.0f ? ((1.0f - qp[s]) - fminf(anr[s], kAlphaMax)) * dal[s] : 0.0f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float4 W = Wv[s];
                const float h = G[s] * fmaf(dap[s], Ov[s].y, dan[s] * Ov[s].x);  // G dL/dG
                const float v1 = fmaf(lyt, W.y, lxt * W.x), v2 = fmaf(lyt, W.w, lxt * W.z);
                // the six pairs and their first halving (row_ror:8): a lane
                // keeps the second value of a pair where bit 3 is set
                const float pa = b3 ? v2 : v1, pb = b3 ? v1 : v2;
                const float ha = h * pa, hb = h * pb, hab = ha * pb;
                const float da = b3 ? dap[s] : dan[s], db = b3 ? dan[s] : dap[s];
                float A[6];
                A[0] = fmaf(h, pa, dpp_move<0x128>(hb));                            // P'_1, P'_2
                A[1] = fmaf(ha, pa, dpp_move<0x128>(hb * pb));                      // Q'_11, Q'_22
                A[2] = halve_l8(hab, h);                                            // Q'_12, S
                A[3] = fmaf(G[s], da, dpp_move<0x128>(G[s] * db));                  // dL/dA_n, dL/dA_p
                A[4] = fmaf(aT[s], ga, dpp_move<0x128>(aT[s] * gb));                // colour 0, 1
                if constexpr (DT) {  // colour 2, dL/dt
                    A[5] = halve_l8(aT[s] * g2, dt[s]);
                } else {
                    A[5] = fmaf(aT[s], g2a, dpp_move<0x128>(aT[s] * g2b));
                }
                float tot = row_reduce12(A, lane);
                // formed by every lane here, where the lane exchange folds into
                // the add, not under the mask of the lanes that hold a slot
                asm volatile("" : "+v"(tot));
                if (slot >= 0) {
                    if constexpr (DET) {
                        if (off[s] != kDead) s_gr[4 * w + q][off[s] / kRec][slot] = tot;
                    } else {
                        if (tot != 0.0f) unsafeAtomicAdd(&rec_at(off[s]).g[slot], (double)tot);
                    }
                }
            }
        }
        __syncthreads();
        // flush: one lane per splat turns the tile's partial sums into the
        // 11 screen-space terms (FP64); then the terms of all splats go out
        // as consecutive atomics, row by row
        if (const int j = PER * w + lane; lane < PER && j < cnt) {  // the entries this wave staged
            Rec &sr = rec_at(kRec * (uint32_t)j);
            double g[kG];
            if constexpr (DET) {
#pragma unroll
                for (int k = 0; k < kG; ++k) g[k] = 0.0;
                for (int row = 0; row < 4 * NW; ++row)  // quarters in a fixed order
#pragma unroll
                    for (int k = 0; k < kG; ++k) g[k] += (double)s_gr[row][j][k];
            } else {
#pragma unroll
                for (int k = 0; k < kG; ++k) g[k] = sr.g[k];
            }
            // moments on the splat's axes about the tile's centre, then about the splat's
            const float4 W = sr.w;
            const double2 cr = s_ref[j];
            const double S = g[5];
            const double P1 = g[0], P2 = g[1], Q11 = g[2], Q22 = g[3], Q12 = g[4];
            const double P[2] = {P1 + cr.x * S, P2 + cr.y * S};
            const double Q[3] = {Q11 + 2.0 * cr.x * P1 + cr.x * cr.x * S,
                                 Q12 + cr.x * P2 + cr.y * P1 + cr.x * cr.y * S,
                                 Q22 + 2.0 * cr.y * P2 + cr.y * cr.y * S};
            double sc[5];
            screen_grad(W, P, Q, sc);
            double dd[11];
#pragma unroll
            for (int k = 0; k < 5; ++k) dd[k] = sc[k];
#pragma unroll
            for (int k = 5; k < 11; ++k) dd[k] = g[k + 1];
            if constexpr (DET) {
                double *o = det.part + (size_t)s_pq[j] * 11;
#pragma unroll
                for (int k = 0; k < 11; ++k) o[k] = dd[k];
            } else {
#pragma unroll
                for (int k = 0; k < 11; ++k) sr.g[k] = dd[k];
            }
        }
        __syncthreads();
        if constexpr (!DET) {
            for (int idx = threadIdx.x; idx < cnt * 11; idx += NT) {
                const int j = idx / 11, k = idx - 11 * j;
                const double val = rec_at(kRec * (uint32_t)j).g[k];
                if (val != 0.0) unsafeAtomicAdd(&sgrad[(size_t)s_id[j] * kG + k], val);
            }
            __syncthreads();
        }
        hi = lo;
    }
    if (lane == 0) wstats[(size_t)tslot * NW + w] = make_uint4(n_eval, n_eval_t, n_con, 0u);
}
template <int TW, int TH, bool DT, bool PERSIST, bool DET>
__global__ __launch_bounds__(TW *TH) void k_blend_bwd(const DevView *__restrict__ views, int nv,
                                                      const uint32_t *__restrict__ tile_order,
                                                      const uint2 *__restrict__ ranges,
                                                      const uint32_t *__restrict__ pair_vals,
                                                      const SplatRec *__restrict__ recs,
                                                      const double4 *__restrict__ axes,
                                                      const float *__restrict__ T_final,
                                                      const uint32_t *__restrict__ n_last,
                                                      const uint8_t *__restrict__ qbits, uint32_t qstride,
                                                      const uint32_t *__restrict__ vis_rank,
                                                      double *__restrict__ sgrad, const DetArgs det,
                                                      uint4 *__restrict__ wstats, uint32_t n_tiles,
                                                      uint32_t *__restrict__ queue, uint32_t chunk)
{
    if constexpr (!PERSIST) {
        blend_bwd_tile<TW, TH, DT, DET>(views, nv, tile_order, ranges, pair_vals, recs, axes, T_final,
                                               n_last, qbits, qstride, vis_rank, sgrad, det, wstats, blockIdx.x);
    } else {
        __shared__ uint32_t s_slot;
        for (;;) {
            const uint32_t first = next_run(queue, chunk, &s_slot);
            if (first >= n_tiles) break;
            const uint32_t last = min(n_tiles, first + chunk);
            for (uint32_t slot = first; slot < last; ++slot) {
                blend_bwd_tile<TW, TH, DT, DET>(views, nv, tile_order, ranges, pair_vals, recs, axes,
                                                       T_final, n_last, qbits, qstride, vis_rank, sgrad, det, wstats,
                                                       slot);
                __syncthreads();  // LDS of this tile read by every wave before the next stages
            }
        }
    }
}

__device__ __forceinline__ void stats_reduce(const uint4 *__restrict__ s, uint32_t n,
                                             unsigned long long *__restrict__ out)
{
    __shared__ unsigned long long s_p[4][3];
    unsigned long long a = 0, b = 0, c = 0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        const uint4 v = s[i];
        a += v.x;
        b += v.y;
        c += v.z;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d, 64);
        b += __shfl_xor(b, d, 64);
        c += __shfl_xor(c, d, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_p[w][0] = a;
        s_p[w][1] = b;
        s_p[w][2] = c;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const unsigned long long t = s_p[0][threadIdx.x] + s_p[1][threadIdx.x] + s_p[2][threadIdx.x] +
                                     s_p[3][threadIdx.x];
        if (t) atomicAdd(&out[threadIdx.x], t);
    }
}

__global__ __launch_bounds__(256) void k_stats_reduce(const uint4 *__restrict__ s, uint32_t n,
                                                      unsigned long long *__restrict__ out)
{
    stats_reduce(s, n, out);
}

// Behind the forward: its counts, and the infinite colours.  The forward adds
// every splat's colour to every pixel, at weight 0 where it does not blend it,
// and 0 inf would be NaN there: an infinite colour stands in its record as -0,
// and goes here to the pixels that blended it (up to its last contributor a
// pixel blends whatever reaches the least alpha).  A wave per 8x8 block; only
// in renders that have such a colour.  (With the forward's sums under the mask
// of the lanes that blend, single frames took 2% longer; with a second form of
// its walk for such renders 16x16 tiles took 3% longer, for their registers.)
__global__ __launch_bounds__(256) void k_blend_end(const uint4 *__restrict__ s, uint32_t n,
                                                   unsigned long long *__restrict__ out,
                                                   const uint32_t *__restrict__ inf_colour,
                                                   const DevView *__restrict__ views, int nv, uint32_t n_tiles,
                                                   const uint2 *__restrict__ ranges,
                                                   const uint32_t *__restrict__ pair_vals,
                                                   const SplatRec *__restrict__ recs,
                                                   const double4 *__restrict__ axes,
                                                   const uint32_t *__restrict__ n_last, int tw, int th)
{
    stats_reduce(s, n, out);
    if (*inf_colour == 0u) return;
    const int lane = threadIdx.x & 63, bx = quarter_x(lane), by = quarter_y(lane);
    const uint32_t nb = (uint32_t)(tw * th / 64), sx = (uint32_t)(tw / 8);
#pragma unroll 1
    for (uint32_t job = blockIdx.x * 4u + (threadIdx.x >> 6); job < n_tiles * nb; job += gridDim.x * 4u) {
        const uint32_t tile = job / nb, bk = job % nb;
        const DevView &V = views[view_of_tile(views, nv, tile)];
        const uint32_t lt = tile - V.tile_base;
        const int ox = (int)(lt % (uint32_t)V.tiles_x) * tw + (int)(bk % sx) * 8;
        const int oy = (int)(lt / (uint32_t)V.tiles_x) * th + (int)(bk / sx) * 8;
        const int px = ox + bx, py = oy + by;
        const bool inside = px < V.W && py < V.H;
        const size_t p = (size_t)py * V.W + px;
        const uint32_t last = inside ? n_last[(size_t)V.pix_base + p] : 0u;
        const uint2 rg = ranges[tile];
#pragma unroll 1
        for (uint32_t i0 = rg.x; i0 < rg.y; i0 += 64) {
            bool marked = false;
            if (i0 + (uint32_t)lane < rg.y) {
                const SplatRec &r = recs[pair_vals[i0 + (uint32_t)lane]];
                marked = signbit(r.r) || signbit(r.g) || signbit(r.b);
            }
            for (uint64_t m = __ballot(marked); m; m &= m - 1ull) {
                const uint32_t i = i0 + (uint32_t)__builtin_ctzll(m), sidx = pair_vals[i];
                const SplatRec r = recs[sidx];
                const double4 W = axes[sidx];
                float c1, c2, d0, d1;
                block_offsets(r, W, ox, oy, c1, c2, d0, d1);
                const float G = eval_gauss(make_float4((float)W.x, (float)W.y, (float)W.z, (float)W.w),
                                           make_float2(c1, c2), (float)bx, (float)by);
                float q, a = fminf(r.An * G, kAlphaMax);
                if (r.t > 0.0f) a = eval_interp(a, 1.0f - fminf(r.Ap * G, kAlphaMax), 1.0f - r.t, r.t, r.invK, q);
                if (a < kAlphaMin || i - rg.x >= last) continue;
                float *o = V.out_rgb + 3 * p;
                if (signbit(r.r)) o[0] = __builtin_inff();
                if (signbit(r.g)) o[1] = __builtin_inff();
                if (signbit(r.b)) o[2] = __builtin_inff();
            }
        }
    }
}

// Workgroups of `kernel` that the whole chip holds at once (CUs times the
// occupancy at `threads` per workgroup): the grid of a persistent launch.
// Looked up once per kernel.
template <typename K>
uint32_t resident_grid(K kernel, int threads)
{
    static std::mutex mu;
    static std::map<const void *, uint32_t> cache;
    std::lock_guard<std::mutex> lock(mu);
    const void *key = reinterpret_cast<const void *>(kernel);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int dev = 0, cus = 0, per = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0);
    const uint32_t g = (uint32_t)std::max(1, std::max(cus, 1) * std::max(per, 1));
    cache[key] = g;
    return g;
}

// Slots per queue ticket of a persistent launch of g workgroups over
// n_tiles slots: about a sixteenth of each workgroup's share, so that the
// last tickets still spread over the grid, and at most 32.
uint32_t queue_run(uint32_t n_tiles, uint32_t g)
{
    const uint32_t share = n_tiles / std::max(g, 1u);
    return std::min(32u, std::max(1u, share / 16u));
}

template <int TW, int TH>
void launch_blend_t(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *order, const uint2 *ranges,
                    const uint32_t *pair_vals, const SplatRec *recs, const double4 *axes, float *T_final,
                    uint32_t *n_last, uint32_t *n_blend, uint8_t *qbits, uint32_t qstride, uint4 *wstats,
                    bool persist, uint32_t *queue, hipStream_t st)
{
    if (persist) {
        auto k = k_blend<TW, TH, true>;
        const uint32_t g = std::min(n_tiles, resident_grid(k, TW * TH));
        launch_fill_u32(queue, 0u, 1, st);
        hipLaunchKernelGGL(k, dim3(g), dim3(TW * TH), 0, st, views, nv, order, ranges, pair_vals, recs, axes,
                           T_final, n_last, n_blend, qbits, qstride, wstats, n_tiles, queue, queue_run(n_tiles, g));
    } else {
        hipLaunchKernelGGL((k_blend<TW, TH, false>), dim3(n_tiles), dim3(TW * TH), 0, st, views, nv, order,
                           ranges, pair_vals, recs, axes, T_final, n_last, n_blend, qbits, qstride, wstats, n_tiles,
                           queue, 1u);
    }
}

template <int TW, int TH, bool DT>
void launch_blend_bwd_dt(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *order, const uint2 *ranges,
                         const uint32_t *pair_vals, const SplatRec *recs, const double4 *axes, const float *T_final,
                         const uint32_t *n_last, const uint8_t *qbits, uint32_t qstride, const uint32_t *vis_rank,
                         double *sgrad, const DetArgs *det, uint4 *wstats, bool persist, uint32_t *queue,
                         hipStream_t st)
{
    if (det) {  // the deterministic mode: one workgroup per tile
        hipLaunchKernelGGL((k_blend_bwd<TW, TH, DT, false, true>), dim3(n_tiles), dim3(TW * TH), 0, st, views, nv,
                           order, ranges, pair_vals, recs, axes, T_final, n_last, qbits, qstride, vis_rank, sgrad,
                           *det, wstats, n_tiles, queue, 1u);
    } else if (persist) {
        auto k = k_blend_bwd<TW, TH, DT, true, false>;
        const uint32_t g = std::min(n_tiles, resident_grid(k, TW * TH));
        launch_fill_u32(queue, 0u, 1, st);
        hipLaunchKernelGGL(k, dim3(g), dim3(TW * TH), 0, st, views, nv, order, ranges, pair_vals, recs, axes, T_final,
                           n_last, qbits, qstride, vis_rank, sgrad, DetArgs{}, wstats, n_tiles, queue,
                           queue_run(n_tiles, g));
    } else {
        hipLaunchKernelGGL((k_blend_bwd<TW, TH, DT, false, false>), dim3(n_tiles), dim3(TW * TH), 0, st, views, nv,
                           order, ranges, pair_vals, recs, axes, T_final, n_last, qbits, qstride, vis_rank, sgrad,
                           DetArgs{}, wstats, n_tiles, queue, 1u);
    }
}

template <int TW, int TH>
void prepare_t()
{
    (void)resident_grid(k_blend<TW, TH, true>, TW * TH);
    (void)resident_grid(k_blend_bwd<TW, TH, true, true, false>, TW * TH);
    (void)resident_grid(k_blend_bwd<TW, TH, false, true, false>, TW * TH);
}

}  // namespace

#define HGS_TILES(X) X(8, 8) X(16, 8) X(16, 16) X(32, 16)

void blend_prepare(int tw, int th)
{
#define X(a, b) \
    if (tw == a && th == b) return prepare_t<a, b>();
    HGS_TILES(X)
#undef X
}

// Supported (tile, batch) combinations; batch 0 means one record per thread.
// A batch above that is accepted and staged one record per thread at a time:
// the records of a larger one keep tiles off the CU (32 views of 1920x1080
// over 30M leaves, forward: 8x8 tiles 4.1 ms with 64, 5.7 with 128, 8.8 with
// 256 records; 16x8 tiles 4.3 ms with 128, 6.2 with 256).  The backward
// stages 32 per wave (64: 7.6 -> 8.9 ms with 16x8 tiles).
bool blend_supported(int tw, int th, int batch)
{
    if (batch == 0) batch = tw * th;
    static constexpr int kCases[][3] = {{8, 8, 64},   {8, 8, 128},    {8, 8, 256},    {16, 8, 128},
                                        {16, 8, 256}, {16, 16, 256}, {16, 16, 512}, {32, 16, 512}};
    for (const int *c : kCases)
        if (tw == c[0] && th == c[1] && batch == c[2]) return true;
    return false;
}

void launch_blend(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *order, const uint2 *ranges,
                  const uint32_t *pair_vals, const SplatRec *recs, const double4 *axes, float *T_final,
                  uint32_t *n_last, uint32_t *n_blend, uint8_t *qbits, uint32_t qstride, uint4 *wstats,
                  Counters *ctr, int tw, int th, bool persist, uint32_t *queue, hipStream_t st)
{
    if (!n_tiles) return;
#define X(a, b)                                                                                                 \
    if (tw == a && th == b)                                                                                     \
        launch_blend_t<a, b>(views, nv, n_tiles, order, ranges, pair_vals, recs, axes, T_final, n_last, n_blend, \
                             qbits, qstride, wstats, persist, queue, st);
    HGS_TILES(X)
#undef X
    hipLaunchKernelGGL(k_blend_end, dim3(256), dim3(256), 0, st, wstats, n_tiles * (uint32_t)(tw * th / 64),
                       &ctr->evaluated, &ctr->inf_colour, views, nv, n_tiles, ranges, pair_vals, recs, axes, n_last, tw,
                       th);
}

void launch_blend_backward(const DevView *views, int nv, uint32_t n_tiles, const uint32_t *order,
                           const uint2 *ranges, const uint32_t *pair_vals, const SplatRec *recs, const double4 *axes,
                           const float *T_final, const uint32_t *n_last, const uint8_t *qbits, uint32_t qstride,
                           const uint32_t *vis_rank, double *sgrad, const DetArgs *det, uint4 *wstats, Counters *ctr,
                           int tw, int th, bool want_dt, bool persist, uint32_t *queue, hipStream_t st)
{
    if (!n_tiles) return;
#define X(a, b)                                                                                                    \
    if (tw == a && th == b) {                                                                                      \
        auto f = want_dt ? launch_blend_bwd_dt<a, b, true> : launch_blend_bwd_dt<a, b, false>;                     \
        f(views, nv, n_tiles, order, ranges, pair_vals, recs, axes, T_final, n_last, qbits, qstride, vis_rank,     \
          sgrad, det, wstats, persist, queue, st);                                                                 \
    }
    HGS_TILES(X)
#undef X
    hipLaunchKernelGGL(k_stats_reduce, dim3(256), dim3(256), 0, st, wstats, n_tiles * (uint32_t)(tw * th / 64),
                       &ctr->bwd_evaluated);
}

}  // namespace hgs
