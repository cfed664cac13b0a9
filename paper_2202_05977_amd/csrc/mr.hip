// Multi-resolution reconstruction (Sec. 5.2): the irradiance is filtered
// at several resolutions, each level with its own predicted weight maps,
// and adjacent levels are blended from the coarsest with Eq. 7:
//   o_p = i^f_p - alpha_p [U D i^f]_p + alpha_p [U i^c]_p
// (D: 2x2 mean, U: nearest-neighbour upsampling).  The per-level filtering
// is the weight-sharing decode (decode.hip, tensor form); this file holds
// the 2x2 mean of the irradiance and the blend.
#include "wskp_internal.h"

namespace wskp {

constexpr int kMrThreads = 256;

// out [H/2, W/2, 3] = 2x2 means of in [H, W, 3] (H, W even)
__global__ __launch_bounds__(kMrThreads) void pool2_kernel(int H, int W, const float *in, float *out)
{
    const int Hc = H / 2, Wc = W / 2;
    const int p = blockIdx.x * kMrThreads + threadIdx.x;
    if (p >= Hc * Wc) return;
    const int y = p / Wc, x = p - y * Wc;
    const float *a = in + ((size_t)(2 * y) * W + 2 * x) * 3;
    const float *b = a + (size_t)W * 3;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
        gstore(out + (size_t)p * 3 + ch,
               0.25f * (((gload(a + ch) + gload(a + 3 + ch)) + gload(b + ch)) + gload(b + 3 + ch)));
}

// One thread per 2x2 block of fine pixels: the block's mean of the fine
// image is formed once and serves its four outputs.  mod (optional)
// remodulates the result.  The four outputs are stored after all loads,
// each pixel's three channels in consecutive stores, so that the L2
// receives whole lines rather than parts of them spread over the kernel.
__global__ __launch_bounds__(kMrThreads) void mr_blend_kernel(int H, int W, const float *fine, const float *coarse,
                                                               const float *alpha, const float *mod, float *out)
{
    const int Hc = H / 2, Wc = W / 2;
    const int p = blockIdx.x * kMrThreads + threadIdx.x;
    if (p >= Hc * Wc) return;
    const int y = p / Wc, x = p - y * Wc;
    size_t q[4];
    q[0] = (size_t)(2 * y) * W + 2 * x;
    q[1] = q[0] + 1;
    q[2] = q[0] + W;
    q[3] = q[2] + 1;
    float f[4][3], a[4], c[3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[k] = gload(alpha + q[k]);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) f[k][ch] = gload(fine + q[k] * 3 + ch);
    }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) c[ch] = gload(coarse + (size_t)p * 3 + ch);
    float o[4][3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float df = 0.25f * (((f[0][ch] + f[1][ch]) + f[2][ch]) + f[3][ch]);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k][ch] = f[k][ch] - a[k] * df + a[k] * c[ch];
    }
    if (mod) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) o[k][ch] *= gload(mod + q[k] * 3 + ch);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) gstore(out + q[k] * 3 + ch, o[k][ch]);
}

// Every blend of the reconstruction in one launch, one thread per 2x2 block
// of finest pixels: the chain of coarser blends that reaches the block's
// coarse pixel (per level four filtered values and one weight) is evaluated
// by each thread that needs it, so no blended image but the result is written.
// The operations of each level are mr_blend_kernel's.  720p, 3 levels: 8.1 us
// in one launch instead of 8.4 + 3.4 in two.
struct MrBlendArgs {
    int H, W;
    const float *f[kMaxLevels], *alpha[kMaxLevels];
    const float *mod;
    float *out;
};
template <int L>
__global__ __launch_bounds__(kMrThreads) void mr_blend_all_kernel(MrBlendArgs m)
{
    const int Hc = m.H / 2, Wc = m.W / 2;
    const int p = blockIdx.x * kMrThreads + threadIdx.x;
    if (p >= Hc * Wc) return;
    const int y = p / Wc, x = p - y * Wc;
    float c[3];
    load_floats<3>(m.f[L - 1] + ((size_t)(y >> (L - 2)) * (m.W >> (L - 1)) + (x >> (L - 2))) * 3, c);
    // the finest level's values, two adjacent pixels at a time
    const size_t q = (size_t)(2 * y) * m.W + 2 * x;
    float f0[2][6], a0[2][2], md[2][6];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        load_floats<6>(m.f[0] + (q + (size_t)r * m.W) * 3, f0[r]);
        load_floats<2>(m.alpha[0] + q + (size_t)r * m.W, a0[r]);
        if (m.mod) load_floats<6>(m.mod + (q + (size_t)r * m.W) * 3, md[r]);
    }
#pragma unroll
    for (int l = L - 2; l >= 1; --l) {
        const int py = y >> (l - 1), px = x >> (l - 1), Wl = m.W >> l;
        const float a = gload(m.alpha[l] + (size_t)py * Wl + px);
        float f[2][6];
#pragma unroll
        for (int r = 0; r < 2; ++r) load_floats<6>(m.f[l] + ((size_t)((py & ~1) + r) * Wl + (px & ~1)) * 3, f[r]);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const float df = 0.25f * (((f[0][ch] + f[0][3 + ch]) + f[1][ch]) + f[1][3 + ch]);
            const float r0 = (px & 1) ? f[0][3 + ch] : f[0][ch], r1 = (px & 1) ? f[1][3 + ch] : f[1][ch];
            const float own = (py & 1) ? r1 : r0;
            c[ch] = own - a * df + a * c[ch];
        }
    }
    float o[2][6];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float df = 0.25f * (((f0[0][ch] + f0[0][3 + ch]) + f0[1][ch]) + f0[1][3 + ch]);
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int k = 0; k < 2; ++k) o[r][3 * k + ch] = f0[r][3 * k + ch] - a0[r][k] * df + a0[r][k] * c[ch];
    }
    if (m.mod) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int k = 0; k < 6; ++k) o[r][k] *= md[r][k];
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) store_floats<6>(m.out + (q + (size_t)r * m.W) * 3, o[r]);
}

hipError_t launch_mr_blend_all(int L, int H, int W, const float *const *f, const float *const *alpha,
                               const float *mod, float *out, hipStream_t s)
{
    MrBlendArgs m{};
    m.H = H;
    m.W = W;
    m.mod = mod;
    m.out = out;
    for (int l = 0; l < L; ++l) {
        m.f[l] = f[l];
        m.alpha[l] = l + 1 < L ? alpha[l] : nullptr;
    }
    const dim3 grid(((H / 2) * (W / 2) + kMrThreads - 1) / kMrThreads), block(kMrThreads);
    switch (L) {
    case 2: hipLaunchKernelGGL(mr_blend_all_kernel<2>, grid, block, 0, s, m); break;
    case 3: hipLaunchKernelGGL(mr_blend_all_kernel<3>, grid, block, 0, s, m); break;
    case 4: hipLaunchKernelGGL(mr_blend_all_kernel<4>, grid, block, 0, s, m); break;
    case 5: hipLaunchKernelGGL(mr_blend_all_kernel<5>, grid, block, 0, s, m); break;
    case 6: hipLaunchKernelGGL(mr_blend_all_kernel<6>, grid, block, 0, s, m); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_pool2(int H, int W, const float *in, float *out, hipStream_t s)
{
    const int n = (H / 2) * (W / 2);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pool2_kernel, dim3((n + kMrThreads - 1) / kMrThreads), dim3(kMrThreads), 0, s, H, W, in,
                       out);
    return hipGetLastError();
}

hipError_t launch_mr_blend(int H, int W, const float *fine, const float *coarse, const float *alpha,
                           const float *mod, float *out, hipStream_t s)
{
    const int n = (H / 2) * (W / 2);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(mr_blend_kernel, dim3((n + kMrThreads - 1) / kMrThreads), dim3(kMrThreads), 0, s, H, W,
                       fine, coarse, alpha, mod, out);
    return hipGetLastError();
}

}  // namespace wskp
