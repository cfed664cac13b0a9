// One training step of the network (Eq. 1: the network's parameters are
// fitted by minimising a loss between the reconstruction and the reference;
// Eq. 6: the SMAPE loss; Sec. 5.3: Adam), FP32 throughout.
//
// The forward pass is the fp32 denoising path (its workspace keeps every
// layer's output).  The backward pass (the frames of one size together):
//   SMAPE gradient at the output -> adjoint of decode and fusion, with the
//   derivative of the weight activation (decode.hip) -> for each conv, from the
//   head back to the first encoder: the weight and bias gradient (accumulated
//   over the frames of the batch) and the input gradient, whose epilogue takes
//   it through the adjoint of the nearest x2 upsampling and the concatenation,
//   or of the 2x2 mean, to the layers that fed the conv (conv_split.hip).  The
//   epilogue that writes the last contribution to an activation's gradient also
//   applies that activation's ReLU mask, and the first contribution
//   overwrites, so no input gradient is stored as such, no gradient buffer
//   cleared and no mask pass run: a step of 8 crops of 256x256, 4 levels, took
//   2477 us with an adjoint and a mask pass per conv and takes 2240.
// The weight gradient's input is written out where it is computed (the
// network input, a 2x2 mean); a decoder's, the [upsampled, skip]
// concatenation, is read from its two sources.  Frames of one size run the
// backward pass together: every kernel once per layer over all of them.
//
// Gradient kernels (NHWC fp32, zero padding, conv = 3x3 cross-correlation):
//   dgrad  gin[p][ci] = sum_{tap,co} gm[p - off(tap)][co] w[co][ci][tap]:
//          itself a 3x3 conv of gm with the kernel flipped and its channel
//          axes swapped, run by the split conv kernel (conv_split.hip) on
//          weights that conv_pack_kernel lays out for it; the head's 2M
//          output channels are padded with zeros to a multiple of 16 (its
//          gradient dh is written with that row stride)
//   wgrad  dw[co][ci][tap] = sum_p gm[p][co] in[p + off(tap)][ci],
//          db[co] = sum_p gm[p][co]: a GEMM over pixels, train_wgrad.hip;
//          each workgroup sums one strip of pixels and a second pass adds
//          the strips' partial sums in a fixed order, so the result does
//          not depend on scheduling
#include "wskp_internal.h"

namespace wskp {

constexpr int kTrThreads = 256;

static inline int tr_blocks(long n) { return (int)((n + kTrThreads - 1) / kTrThreads); }

// The per-frame kernels below run over a group of frames (blockIdx.y), the
// frames' own buffers passed by pointer (TrFrames) and the group's scratch
// contiguous per frame.

// network input X [P][10] (Sec. 5.1), as the first conv's staging forms it
__global__ __launch_bounds__(kTrThreads) void tr_pack_kernel(long P, TrFrames fr, float inv_gamma, float dnear,
                                                              float dinv, float *X)
{
    const long p = (long)blockIdx.x * kTrThreads + threadIdx.x;
    if (p >= P) return;
    const int f = blockIdx.y;
    const float *r = fr.r[f], *a = fr.a[f], *n = fr.n[f], *d = fr.d[f];
    X += f * P * 10;
    float x[10];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float rv = fminf(fmaxf(gload(r + p * 3 + ch), 0.f), 1.f);
        x[ch] = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(rv) * inv_gamma);
        x[3 + ch] = gload(a + p * 3 + ch);
        x[6 + ch] = (gload(n + p * 3 + ch) + 1.f) * 0.5f;
    }
    x[9] = fminf(fmaxf((gload(d + p) - dnear) * dinv, 0.f), 1.f);
#pragma unroll
    for (int ch = 0; ch < 10; ++ch) gstore(X + p * 10 + ch, x[ch]);
}

// Kernels over nf frames of one size: frame f's operand X sits at X + f sX
// (floats); outputs are contiguous per frame.

// out [nf][H/2][W/2][C] = 2x2 means of in [H][W][C] (frame stride sin)
__global__ __launch_bounds__(kTrThreads) void tr_pool_kernel(int H, int W, int C, int nf, const float *in, long sin,
                                                              float *out)
{
    const int Wo = W / 2;
    const long n = (long)(H / 2) * Wo * C;
    const long i = (long)blockIdx.x * kTrThreads + threadIdx.x;
    if (i >= n * nf) return;
    const long f = i / n, j = i - f * n;
    const int ch = (int)(j % C);
    const long q = j / C;
    const int y = (int)(q / Wo), x = (int)(q % Wo);
    const float *s = in + f * sin + ((long)(2 * y) * W + 2 * x) * C + ch;
    gstore(out + i, 0.25f * (((gload(s) + gload(s + C)) + gload(s + (long)W * C)) + gload(s + (long)W * C + C)));
}

// interleaved head [P][2M] from the planar record [2M][P]; c = r/(a+eps_a),
// mod = a + eps_a (the decode adjoint's inputs)
// (whole records and pixels per store: one float per store, 8 M bytes apart
// across lanes, took 36 us for 8 crops of 256x256; now 14)
template <int M>
__global__ __launch_bounds__(kTrThreads) void tr_head_prep_kernel(long P, const float *planar, long sp, TrFrames fr,
                                                                   float eps_a, float *head, float *c, float *mod)
{
    const long p = (long)blockIdx.x * kTrThreads + threadIdx.x;
    if (p >= P) return;
    const int f = blockIdx.y;
    float rec[2 * M], r[3], a[3];
    load_floats<3>(fr.r[f] + p * 3, r);
    load_floats<3>(fr.a[f] + p * 3, a);
#pragma unroll
    for (int j = 0; j < 2 * M; ++j) rec[j] = gload(planar + f * sp + (long)j * P + p);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        a[ch] += eps_a;
        r[ch] /= a[ch];
    }
    store_floats<2 * M>(head + (f * P + p) * 2 * M, rec);
    store_floats<3>(mod + (f * P + p) * 3, a);
    store_floats<3>(c + (f * P + p) * 3, r);
}

// SMAPE (Eq. 6) gradient g = dL/dy for n values of each frame with mean
// weight inv_n, and the block's share of the loss in
// partial[frame * gridDim.x + blockIdx.x]
__global__ __launch_bounds__(kTrThreads) void tr_smape_kernel(long n, TrFrames fr, float eps, float inv_n, float *g,
                                                               float *partial)
{
    __shared__ float red[kTrThreads];
    const long i = (long)blockIdx.x * kTrThreads + threadIdx.x;
    const int f = blockIdx.y;
    const float *y = fr.y[f], *t = fr.t[f];
    g += f * n;
    partial += (long)f * gridDim.x;
    float l = 0.f;
    if (i < n) {
        const float yv = gload(y + i), tv = gload(t + i);
        const float d = yv - tv, den = fabsf(yv) + fabsf(tv) + eps;
        const float sd = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
        const float sr = yv > 0.f ? 1.f : (yv < 0.f ? -1.f : 0.f);
        l = fabsf(d) / den;
        gstore(g + i, (sd * den - fabsf(d) * sr) / (den * den) * inv_n);
    }
    red[threadIdx.x] = l;
    __syncthreads();
    for (int s = kTrThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) gstore(partial + blockIdx.x, red[0] * inv_n);
}

// loss[0] (+)= sum of partial[0..nb): thread i sums partial[i], [i + 256],
// ... in order, then the 256 sums are added pairwise in LDS (a fixed order)
__global__ __launch_bounds__(kTrThreads) void tr_sum_kernel(int nb, const float *partial, float *loss, int accumulate)
{
    __shared__ float red[kTrThreads];
    float v = 0.f;
    for (int b = threadIdx.x; b < nb; b += kTrThreads) v += gload(partial + b);
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = kTrThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) gstore(loss, (accumulate ? gload(loss) : 0.f) + red[0]);
}

// First level of a sliced reduce: out[y][i] = sum of part rows (chunks)
// y S .. y S + S - 1 (fixed order: four interleaved sums added pairwise), for
// the nw weights then the Co biases; blockIdx.y = slice y.  Used when a layer
// has few weights and many chunks, so that more workgroups share the sums.
__global__ __launch_bounds__(kTrThreads) void tr_wgrad_slice_kernel(long nw, int Co, int nchunk, int S,
                                                                     const float *part, const float *partb,
                                                                     float *out)
{
    __shared__ float sred[4][64];
    const int li = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const long i = (long)blockIdx.x * 64 + li;
    const bool inw = i < nw, in = i < nw + Co;
    const float *src = inw ? part + i : partb + (in ? i - nw : 0);
    const long stride = inw ? nw : Co;
    const int c0 = blockIdx.y * S, c1 = min(nchunk, c0 + S);
    float s0 = 0.f;
    if (in)
        for (int c = c0 + grp; c < c1; c += 4) s0 += gload(src + (long)c * stride);
    sred[grp][li] = s0;
    __syncthreads();
    if (grp == 0 && in)
        gstore(out + (long)blockIdx.y * (nw + Co) + i, (sred[0][li] + sred[1][li]) + (sred[2][li] + sred[3][li]));
}

// dw (+)= sum over chunks of part, likewise db: 64 weights per workgroup,
// its four waves take the chunks c = wave (mod 4) and each sums them in
// order on two alternating accumulators; the waves' sums are added in a
// fixed order, so the result does not depend on scheduling
__global__ __launch_bounds__(kTrThreads) void tr_wgrad_reduce_kernel(long nw, int Co, int nchunk, const float *part,
                                                                      const float *partb, float *dw, float *db,
                                                                      int accumulate)
{
    __shared__ float sred[4][64];
    const int li = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const long i = (long)blockIdx.x * 64 + li;
    const bool inw = i < nw, in = i < nw + Co;
    const float *src = inw ? part + i : partb + (in ? i - nw : 0);
    const long stride = inw ? nw : Co;
    float s0 = 0.f, s1 = 0.f;
    if (in) {
        int c = grp;
        for (; c + 4 < nchunk; c += 8) {
            s0 += gload(src + (long)c * stride);
            s1 += gload(src + (long)(c + 4) * stride);
        }
        if (c < nchunk) s0 += gload(src + (long)c * stride);
    }
    sred[grp][li] = s0 + s1;
    __syncthreads();
    if (grp == 0 && in) {
        float *dst = inw ? dw + i : db + (i - nw);
        const float v = (sred[0][li] + sred[1][li]) + (sred[2][li] + sred[3][li]);
        gstore(dst, accumulate ? gload(dst) + v : v);
    }
}

// one thread per (table, frame)
__global__ void tr_frame_tables_kernel(FrameDesc *tab, int nf, TrConvTables tables)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nf * tables.n) return;
    tab[i] = tr_conv_frame(tables.t[i / nf], i % nf);
}

// Adam (Kingma and Ba): m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// w -= lr (m / c1) / (sqrt(v / c2) + eps) with c1 = 1 - b1^t, c2 = 1 - b2^t
__global__ __launch_bounds__(kTrThreads) void tr_adam_kernel(long n, float *w, const float *g, float *m, float *v,
                                                              float lr, float b1, float b2, float c1, float c2,
                                                              float eps)
{
    const long i = (long)blockIdx.x * kTrThreads + threadIdx.x;
    if (i >= n) return;
    const float gi = gload(g + i);
    const float mi = b1 * gload(m + i) + (1.f - b1) * gi;
    const float vi = b2 * gload(v + i) + (1.f - b2) * gi * gi;
    gstore(m + i, mi);
    gstore(v + i, vi);
    gstore(w + i, gload(w + i) - lr * (mi / c1) / (sqrtf(vi / c2) + eps));
}

// ---- launchers ---------------------------------------------------------------
#define TR_LAUNCH(kernel, n, ...)                                                                          \
    do {                                                                                                   \
        const long n_ = (n);                                                                               \
        if (n_ > 0) hipLaunchKernelGGL(kernel, dim3(tr_blocks(n_)), dim3(kTrThreads), 0, s, __VA_ARGS__); \
    } while (0)

// grid of one frame's blocks (x) over the group's nf frames (y)
#define TR_LAUNCH_F(kernel, n, nf, ...)                                                                    \
    do {                                                                                                   \
        const long n_ = (n);                                                                               \
        if (n_ > 0 && (nf) > 0)                                                                            \
            hipLaunchKernelGGL(kernel, dim3(tr_blocks(n_), (unsigned)(nf)), dim3(kTrThreads), 0, s, __VA_ARGS__); \
    } while (0)

hipError_t tr_pack(long P, int nf, const TrFrames &fr, float inv_gamma, float dnear, float dinv, float *X,
                   hipStream_t s)
{
    TR_LAUNCH_F(tr_pack_kernel, P, nf, P, fr, inv_gamma, dnear, dinv, X);
    return hipGetLastError();
}
hipError_t tr_pool(int H, int W, int C, int nf, const float *in, long sin, float *out, hipStream_t s)
{
    TR_LAUNCH(tr_pool_kernel, (long)(H / 2) * (W / 2) * C * nf, H, W, C, nf, in, sin, out);
    return hipGetLastError();
}
hipError_t tr_head_prep(long P, int M, int nf, const float *planar, long sp, const TrFrames &fr, float eps_a,
                        float *head, float *c, float *mod, hipStream_t s)
{
    switch (M) {
#define TR_M(m) \
    case m: TR_LAUNCH_F(tr_head_prep_kernel<m>, P, nf, P, planar, sp, fr, eps_a, head, c, mod); break;
        TR_M(1) TR_M(2) TR_M(3) TR_M(4) TR_M(5) TR_M(6) TR_M(7) TR_M(8)
#undef TR_M
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
int tr_smape_blocks(long n) { return tr_blocks(n); }
hipError_t tr_smape(long n, int nf, const TrFrames &fr, float eps, float inv_n, float *g, float *partial, float *loss,
                    int accumulate, hipStream_t s)
{
    TR_LAUNCH_F(tr_smape_kernel, n, nf, n, fr, eps, inv_n, g, partial);
    hipLaunchKernelGGL(tr_sum_kernel, dim3(1), dim3(kTrThreads), 0, s, tr_blocks(n) * nf, partial, loss, accumulate);
    return hipGetLastError();
}
// slices of the two-level reduce (at most kWgSlices)
constexpr int kWgSlices = 64;
static int wgrad_slices(long nw, int Co, int nall)
{
    const long gx = (nw + Co + 63) / 64;
    int G = 1;
    while (G < kWgSlices && gx * G < 1024 && nall / (2 * G) >= 32) G *= 2;
    return G;
}
size_t tr_wgrad_part_floats(int H, int W, int Ci, int Co, int nf)
{
    // the strips' partial sums, then the slices' sums of the two-level reduce
    return ((size_t)tr_wgrad_strips(H, W, Ci, Co, nf) + kWgSlices) * ((size_t)Co * Ci * 9 + Co);
}
hipError_t tr_wgrad(int H, int W, int Co, int ldg, int nf, const float *gm, long sgm, const float *in, long sin,
                    int Cf, const float *up, long sup, int Cu, float *part, float *dw, float *db, bool accumulate,
                    hipStream_t s)
{
    const int Ci = Cu + Cf, nall = tr_wgrad_strips(H, W, Ci, Co, nf);
    const long nw = (long)Co * Ci * 9;
    float *partb = part + (size_t)nall * nw;
    const hipError_t e = launch_wgrad_split(H, W, Co, ldg, nf, gm, sgm, in, sin, Cf, up, sup, Cu, part, partb, s);
    if (e != hipSuccess) return e;
    const unsigned gx = (unsigned)((nw + Co + 63) / 64);
    // (the second level treats the biases as weights nw .. nw + Co - 1, so
    // db must follow dw, as in the weight blob)
    const int G = db == dw + nw ? wgrad_slices(nw, Co, nall) : 1;
    if (G == 1) {
        hipLaunchKernelGGL(tr_wgrad_reduce_kernel, dim3(gx), dim3(kTrThreads), 0, s, nw, Co, nall, part, partb, dw, db,
                           accumulate ? 1 : 0);
    } else {
        // slice sums into the rows after the chunks' partials, then their sum
        float *sl = partb + (size_t)nall * Co;
        const int S = (nall + G - 1) / G;
        hipLaunchKernelGGL(tr_wgrad_slice_kernel, dim3(gx, (unsigned)G), dim3(kTrThreads), 0, s, nw, Co, nall, S, part,
                           partb, sl);
        // rows of sl are nw + Co floats: weights, then biases
        hipLaunchKernelGGL(tr_wgrad_reduce_kernel, dim3(gx), dim3(kTrThreads), 0, s, nw + Co, 0, G, sl, sl, dw, db,
                           accumulate ? 1 : 0);
    }
    return hipGetLastError();
}
hipError_t tr_frame_tables(FrameDesc *tab, int nf, const TrConvTables &tables, hipStream_t s)
{
    hipLaunchKernelGGL(tr_frame_tables_kernel, dim3((unsigned)((nf * tables.n + 63) / 64)), dim3(64), 0, s, tab, nf,
                       tables);
    return hipGetLastError();
}
hipError_t tr_adam(long n, float *w, const float *g, float *m, float *v, float lr, float b1, float b2, float c1,
                   float c2, float eps, hipStream_t s)
{
    TR_LAUNCH(tr_adam_kernel, n, n, w, g, m, v, lr, b1, b2, c1, c2, eps);
    return hipGetLastError();
}

}  // namespace wskp
