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

// blockIdx.y: the view.  Four values at a time where the view's three arrays
// are 16-byte aligned (each thread one pixel, 4 bytes at a time, and a search
// for its view took 0.55 ms for 16 views of 1920x1080, this 0.23).
__global__ __launch_bounds__(kT) void k_l1(const DevView *__restrict__ views, double inv_m,
                                           double *__restrict__ partial)
{
    __shared__ double s_w[kT / 64];
    const DevView &V = views[blockIdx.y];
    const float *img = V.out_rgb, *ref = V.target;
    float *dl = const_cast<float *>(V.dL);
    const uint32_t n = 3u * (uint32_t)V.W * (uint32_t)V.H;  // images are at most 32768 x 32768
    const uint32_t n4 = (((uintptr_t)img | (uintptr_t)ref | (uintptr_t)dl) & 15u) ? 0u : n / 4u;
    const float m = (float)inv_m;
    double acc = 0.0;
    auto one = [&](float a, float b) -> float {
        const float d = a - b;
        acc += fabs((double)d);
        return d > 0.0f ? m : (d < 0.0f ? -m : 0.0f);
    };
    const uint32_t first = blockIdx.x * kT + threadIdx.x, step = gridDim.x * kT;
    for (uint32_t i = first; i < n4; i += step) {
        const float4 a = reinterpret_cast<const float4 *>(img)[i], b = reinterpret_cast<const float4 *>(ref)[i];
        reinterpret_cast<float4 *>(dl)[i] = make_float4(one(a.x, b.x), one(a.y, b.y), one(a.z, b.z), one(a.w, b.w));
    }
    for (uint32_t i = 4u * n4 + first; i < n; i += step) dl[i] = one(img[i], ref[i]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kT / 64; ++w) t += s_w[w];
        partial[blockIdx.y * gridDim.x + blockIdx.x] = t;
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
    // a workgroup per 1024 values of an average view, kL1Blocks in all
    const uint32_t per = (uint32_t)std::min<uint64_t>((m / nv + 4 * kT - 1) / (4 * kT), kL1Blocks / nv);
    const uint32_t x = std::max(per, 1u);
    hipLaunchKernelGGL(k_l1, dim3(x, nv), dim3(kT), 0, st, views, inv_m, partial);
    hipLaunchKernelGGL(k_l1_final, dim3(1), dim3(kT), 0, st, partial, (int)(x * (uint32_t)nv), inv_m, loss);
}

}  // namespace hgs
