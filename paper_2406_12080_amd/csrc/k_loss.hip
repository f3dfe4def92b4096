// Loss of the hierarchy optimisation (Sec. 5.1 optimises the hierarchy's
// interior nodes against the training images; the loss used here is the
// L1 distance, the image term of 3D Gaussian Splatting's loss): for the
// views of one render,
//   loss = (1 / M) sum over views, pixels and channels |C - C*|,
//   dL/dC = sign(C - C*) / M  (sign(0) = 0),
// with M the number of image values.  HBM-bound: per pixel it reads the
// image and the target and writes the cotangent (36 B).  The sum runs in
// FP64 over fixed per-block partials and one final block, so that it does
// not depend on scheduling.
#include "hgs_internal.h"

namespace hgs {

namespace {

constexpr int kT = 256;

// The pixels of all views one behind the other are cut into runs of kRun, which
// the workgroups take in turn, view by view, four values at a time where the
// view's three arrays are 16-byte aligned: 16 views of 1920x1080 in 0.24 ms
// (each thread one pixel, 4 bytes at a time, and a search for its view: 0.55
// ms; as many workgroups for every view: 0.24 ms, but 1.05 for one view of
// 3840x2160 among 255 of 64x64, which take 0.22 so, the most of it the host's).
constexpr uint32_t kRun = 1024;

__global__ __launch_bounds__(kT) void k_l1(const DevView *__restrict__ views, int nv, uint32_t n_pix, double inv_m,
                                           double *__restrict__ partial)
{
    __shared__ double s_w[kT / 64];
    const float m = (float)inv_m;
    double acc = 0.0;
    auto one = [&](float a, float b) -> float {
        const float d = a - b;
        acc += fabs((double)d);
        return d > 0.0f ? m : (d < 0.0f ? -m : 0.0f);
    };
    int vi = 0;           // the view of pixel g
    uint64_t end = 0ull;  // the first pixel behind it
    for (uint64_t r = (uint64_t)blockIdx.x * kRun; r < n_pix; r += (uint64_t)gridDim.x * kRun) {
        const uint64_t g1 = min(r + kRun, (uint64_t)n_pix);
        for (uint64_t g = r; g < g1;) {
            if (g >= end) {  // the last view that begins at or before g
                vi = -1;
                for (int v0 = 0; v0 < nv; v0 += 64) {
                    const int v = v0 + (int)(threadIdx.x & 63);
                    vi += __popcll(__ballot(v < nv && views[v].pix_base <= g));
                }
            }
            const DevView &V = views[vi];
            end = (uint64_t)V.pix_base + (uint64_t)V.W * (uint64_t)V.H;
            const float *img = V.out_rgb, *ref = V.target;
            float *dl = const_cast<float *>(V.dL);
            // values [a, b) of the view (images are at most 32768 x 32768), of
            // them the vectors [a4, b4)
            const uint32_t a = 3u * (uint32_t)(g - V.pix_base), b = 3u * (uint32_t)(min(end, g1) - V.pix_base);
            const bool aligned = (((uintptr_t)img | (uintptr_t)ref | (uintptr_t)dl) & 15u) == 0u;
            const uint32_t a4 = aligned ? (a + 3u) / 4u : 0u, b4 = aligned ? max(b / 4u, a4) : 0u;
#pragma unroll 3
            for (uint32_t i = a4 + threadIdx.x; i < b4; i += kT) {
                const float4 x = reinterpret_cast<const float4 *>(img)[i], y = reinterpret_cast<const float4 *>(ref)[i];
                reinterpret_cast<float4 *>(dl)[i] =
                    make_float4(one(x.x, y.x), one(x.y, y.y), one(x.z, y.z), one(x.w, y.w));
            }
            const uint32_t head = aligned ? min(4u * a4, b) : b;  // the values before the vectors, and those behind
            for (uint32_t i = a + threadIdx.x; i < head; i += kT) dl[i] = one(img[i], ref[i]);
            for (uint32_t i = max(4u * b4, head) + threadIdx.x; i < b; i += kT) dl[i] = one(img[i], ref[i]);
            g = min(end, g1);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kT / 64; ++w) t += s_w[w];
        partial[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kT) void k_l1_final(const double *__restrict__ partial, int n, double inv_m,
                                                 double *__restrict__ loss)
{
    __shared__ double s_w[kT / 64];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kT) acc += partial[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kT / 64; ++w) t += s_w[w];
        *loss = t * inv_m;
    }
}

}  // namespace

void launch_l1(const DevView *views, int nv, uint32_t n_pix, double *partial, double *loss, hipStream_t st)
{
    const uint64_t m = (uint64_t)n_pix * 3;
    const double inv_m = m ? 1.0 / (double)m : 0.0;
    if (!m || nv <= 0) return;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(((uint64_t)n_pix + kRun - 1) / kRun, kL1Blocks);
    hipLaunchKernelGGL(k_l1, dim3(blocks), dim3(kT), 0, st, views, nv, n_pix, inv_m, partial);
    hipLaunchKernelGGL(k_l1_final, dim3(1), dim3(kT), 0, st, partial, (int)blocks, inv_m, loss);
}

}  // namespace hgs
