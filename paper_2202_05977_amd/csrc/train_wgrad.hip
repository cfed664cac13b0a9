// Weight gradients of the training step on the bf16 matrix cores:
//   dw[co][ci][tap] = sum_p gm[p][co] in[p + off(tap)][ci],  db[co] = sum_p gm[p][co]
// (3x3, zero padding, NHWC fp32), a GEMM over pixels.  Every fp32 operand is
// taken as the sum of three bf16 parts (split_bf16) and a product as its six
// largest part products, the five small ones in an accumulator of their own
// (conv_split.hip: closer to float64 than v_mfma_f32_16x16x4f32, at 2.7 times
// its rate).  Strips with infinite or very large operands are summed again by a
// careful pass (see there), which costs the others nothing: a step of 8 crops of
// 256x256 takes 2166 us without it and 2170 with it, the runs' spread.
//
// A workgroup of 4 waves owns 32 output x 32 input channels, a wave 16 x 16
// with all 9 taps (v_mfma_f32_16x16x32_bf16, 32 pixels of an image row per
// MFMA), over a strip of 32 columns x `rows` rows of one frame.  K runs over
// pixels, but memory holds a pixel's channels together: staging transposes,
// each thread splitting 2 pixels x 4 channels into packed pixel pairs, and LDS
// holds rows [part][channel][pixel].  The strip is walked by input rows: the
// three column offsets of an input row are made in registers from one
// aligned fragment and its neighbours (5 shifts), and serve the taps of the
// three gradient rows that touch the row, whose fragments stay in registers:
// per 54 MFMAs a wave reads 7.5 KiB of LDS.  The next row is written to the other
// LDS buffer and the one after that is in flight while a row's MFMAs run.
//
// Each strip's sums go to `part` and `partb`, which the reduce kernels of
// train.hip add in a fixed order.
//
// Measured, 8 crops of 256x256: 96 -> 32 channels 373 -> 166 us (175 TFLOP/s of
// fp32 work, 1050 of bf16 MFMAs), 160 -> 64 304 -> 145, all eight layers 1187 ->
// 620 us per step.  What bounds it now: MFMA issue (16x16x32 takes 19.5 cycles of
// 16 from two waves per SIMD) and staging, which each of the two layers with
// 10 channels on a side (57 us) is bound by alone.
#include "conv_device.h"

namespace wskp {

constexpr int kWsIn = 112, kWsGm = 80;    // bytes per channel of an LDS row: 48 and 32 pixels, bank-spread
constexpr int kWsInRow = 3 * 32 * kWsIn, kWsGmRow = 3 * 32 * kWsGm;
constexpr unsigned kWsOut = 0x80000000u;  // beyond every buffer (maps stay below 2 GiB): loads read zeros

// VEC: the input's channel counts are multiples of 4 (else the network input's
// 10: one load per channel).
template <bool VEC>
__global__ __launch_bounds__(256, 2) void tr_wgrad_split_kernel(int H, int W, int Co, int ldg, int rows, int strips_x,
                                                                int strips_y, const float *gm, long sgm,
                                                                const float *in, long sin, int Cf, const float *up,
                                                                long sup, int Cu, float *part, float *partb)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[2][kWsInRow + kWsGmRow];
    __shared__ int again;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 15, lq = lane >> 4;
    const int co0 = blockIdx.y * 32, ci0 = blockIdx.z * 32, Ci = Cu + Cf;
    // strip: frame, rows ya .. yb - 1 of the gradient, columns x0 .. x0 + 31
    const int per = strips_x * strips_y;
    const int fr = blockIdx.x / per, st = blockIdx.x - fr * per;
    const int x0 = st % strips_x * 32, ya = st / strips_x * rows, yb = min(H, ya + rows);
    const rsrc_t rg = make_rsrc(gm + fr * sgm, (unsigned)H * W * ldg * 4u);

    // ---- staging items: 2 pixels x 4 channels.  Items 0..127: the gradient
    // row, pixel pair it / 8 (of 16), channels 4 (it % 8) ..; items 128..271:
    // the input row, pixel pair (it - 128) / 8 of the 18 at x0 - 2 .. x0 + 33.
    // A 16-channel half of the input block lies in one source: the H x W map,
    // or the map of half the size that the input upsamples.
    struct Item {
        bool is_in, ok;
        int x, c, Cs, sh, Ws;     // first pixel, channel of its source, the source's channels, shift, width
        int dst;                  // LDS offset of part 0 of the first channel
    };
    auto item = [&](int it) {
        Item r{};
        r.is_in = it >= 128;
        r.ok = it < 272;
        const int j = r.is_in ? it - 128 : it, cg = j & 7, pp = j >> 3;
        if (!r.is_in) {
            r.x = x0 + 2 * pp;
            r.c = co0 + 4 * cg;
            r.Cs = ldg;
            r.Ws = W;
            r.dst = kWsInRow + 4 * cg * kWsGm + 4 * pp;
            r.ok = r.ok && r.c < ldg;
        } else {
            const int ch = ci0 + 4 * cg;
            const bool coarse = ch < Cu;
            r.x = x0 - 2 + 2 * pp;
            r.c = coarse ? ch : ch - Cu;
            r.Cs = coarse ? Cu : Cf;
            r.sh = coarse ? 1 : 0;
            r.Ws = W >> r.sh;
            r.dst = 4 * cg * kWsIn + 12 + 4 * pp;    // (48 pixels from x0 - 8)
            r.ok = r.ok && ch < Ci;
        }
        return r;
    };
    const rsrc_t rin = make_rsrc(in + fr * sin, (unsigned)H * W * Cf * 4u);
    const rsrc_t rup = make_rsrc(Cu ? up + fr * sup : in, Cu ? (unsigned)(H >> 1) * (W >> 1) * Cu * 4u : 0u);
    // item A: tid (gradient for tid < 128, input after); item B: 256 + tid for tid < 16
    const Item ia = item(tid), ib = item(256 + tid);
    float va[2][4], vb[2][4];
    // loads of one item for image row y of the input / the gradient
    auto load_item = [&](const Item &it, int y, float (&v)[2][4]) {
        const bool rok = it.ok && y >= 0 && y < H && (it.is_in || (y >= ya && y < yb));
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int x = it.x + p;
            const bool ok = rok && x >= 0 && x < W;
            const unsigned off = ((unsigned)((y >> it.sh) * it.Ws + (x >> it.sh)) * (unsigned)it.Cs + (unsigned)it.c) * 4u;
            const unsigned o = ok ? off : kWsOut;
            if (VEC || !it.is_in) {
                const gf32x4 q = __builtin_bit_cast(
                    gf32x4, !it.is_in ? __builtin_amdgcn_raw_buffer_load_b128(rg, (int)o, 0, 0)
                                      : (it.sh ? __builtin_amdgcn_raw_buffer_load_b128(rup, (int)o, 0, 0)
                                               : __builtin_amdgcn_raw_buffer_load_b128(rin, (int)o, 0, 0)));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[p][e] = q[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[p][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rin, (int)(it.c + e < it.Cs ? o + 4u * e : kWsOut), 0, 0));
            }
        }
    };
    auto put_item = [&](auto careful, const Item &it, int buf, const float (&v)[2][4]) {
        const int stride = it.is_in ? kWsIn : kWsGm, part_b = it.is_in ? 32 * kWsIn : 32 * kWsGm;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            unsigned p[3];
            split_bf16<careful()>(v[0][e], v[1][e], p);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<unsigned *>(&smem[buf][it.dst + q * part_b + e * stride]) = p[q];
        }
    };
    // step s stages input row ya - 1 + s and gradient row ya + s
    auto fetch = [&](int s) {
        load_item(ia, (ia.is_in ? ya - 1 : ya) + s, va);
        if (wave == 0) load_item(ib, ya - 1 + s, vb);
    };
    auto commit = [&](auto careful, int buf) {
        put_item(careful, ia, buf, va);
        if (tid < 16) put_item(careful, ib, buf, vb);
    };

    // ---- accumulators of 16 co x 16 ci: main and small terms of each tap, and
    // the bias (gradient times one) for input block 0
    const int coh = wave & 1, cih = wave >> 1;
    const bool bias = blockIdx.z == 0 && cih == 0;
    // (a 16 x 16 block past the layer's channels: its wave only stages)
    const bool live = co0 + coh * 16 < Co && ci0 + cih * 16 < Ci;
    f32x4 acc[9], sml[9], bm, bs;
    // gradient fragments of rows y + 1, y, y - 1 of the current input row y
    bf16x8 g[3][3];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] = sml[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        bm = bs = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int q = 0; q < 3; ++q) g[r][q] = __builtin_bit_cast(bf16x8, u16x8{0, 0, 0, 0, 0, 0, 0, 0});
    };
    clear();
    const bf16x8 one = __builtin_bit_cast(
        bf16x8, u16x8{0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80});

    // One pass over the strip.  The careful one takes the wide split, and only rows and
    // columns of the image: elsewhere the gradient is zero, and zero times an
    // infinity or a NaN is NaN.
    const int steps = yb - ya + 2;   // input rows ya - 1 .. yb
    auto strip = [&](auto careful) {
        // (dx = 0) the input beside column W, the image's last, in this lane's dword i
        auto past = [&](int i) {
            const int d = W - x0 - (lq * 8 + 2 * i);
            return d == 0 ? 0xffff0000u : d == 1 ? 0x0000ffffu : 0xffffffffu;
        };
        fetch(0);
        commit(careful, 0);
        fetch(1);
        lds_sync();
        for (int s = 0; s < steps; ++s) {
            const int buf = s & 1;
            const unsigned char *row = smem[buf];
            if (s + 1 < steps) commit(careful, buf ^ 1);   // its loads were issued a step ago
            if (s + 2 < steps) fetch(s + 2);
            if (!live) {
                lds_sync();
                continue;
            }
            // rows roll: g[2] = row y - 1, g[1] = row y, g[0] = row y + 1 (new)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                g[2][q] = g[1][q];
                g[1][q] = g[0][q];
                g[0][q] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const gu32x4 *>(&row[kWsInRow + (q * 32 + coh * 16 + lj) * kWsGm + lq * 16]));
            }
            bf16x8 x[3][3];   // [part][dx]
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const unsigned char *b = &row[(q * 32 + cih * 16 + lj) * kWsIn + 16 + lq * 16];
                const gu32x4 c = *reinterpret_cast<const gu32x4 *>(b);
                const unsigned pv = *reinterpret_cast<const unsigned *>(b - 4), nx = *reinterpret_cast<const unsigned *>(b + 16);
                unsigned s0 = __builtin_amdgcn_alignbit(c[0], pv, 16), s1 = __builtin_amdgcn_alignbit(c[1], c[0], 16);
                unsigned s2 = __builtin_amdgcn_alignbit(c[2], c[1], 16), s3 = __builtin_amdgcn_alignbit(c[3], c[2], 16);
                const unsigned s4 = __builtin_amdgcn_alignbit(nx, c[3], 16);
                x[q][2] = __builtin_bit_cast(bf16x8, gu32x4{s1, s2, s3, s4});
                if constexpr (careful()) {
                    s0 &= past(0);
                    s1 &= past(1);
                    s2 &= past(2);
                    s3 &= past(3);
                }
                x[q][0] = __builtin_bit_cast(bf16x8, gu32x4{s0, s1, s2, s3});
                x[q][1] = __builtin_bit_cast(bf16x8, c);
            }
            // tap (dy, dx) of gradient row y - dy + 1
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                // (gradient part, input part): the smallest products first
                const int gq = k == 0 ? 2 : k == 1 ? 0 : k == 2 ? 1 : k == 3 ? 1 : 0;
                const int xq = k == 0 ? 0 : k == 1 ? 2 : k == 2 ? 1 : k == 3 ? 0 : k == 4 ? 1 : 0;
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    if (careful() && (s < t / 3 || s - t / 3 >= yb - ya)) continue;
                    f32x4 &d = k < 5 ? sml[t] : acc[t];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[t / 3][gq], x[xq][t % 3], d, 0, 0, 0);
                }
            }
            if (bias) {
                bs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[0][2], one, bs, 0, 0, 0);
                bs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[0][1], one, bs, 0, 0, 0);
                bm = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[0][0], one, bm, 0, 0, 0);
            }
            lds_sync();
        }
    };
    if (tid == 0) again = 0;
    strip(std::false_type{});
    // A NaN among the sums is an operand's, or came of an infinite or very large
    // operand: if the strip has one, it is summed again.
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) z += acc[t][r] + sml[t][r];
#pragma unroll
    for (int r = 0; r < 4; ++r) z += bm[r] + bs[r];
    if (z != z) again = 1;
    lds_sync();
    if (__builtin_amdgcn_readfirstlane(again)) {
        float big = 0.f;
        auto note = [&](const Item &it, const float (&v)[2][4]) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    big = fmaxf(big, fabsf(v[p][e]));
                    // (maps other than the network's input hold no NaN: the ReLU drops them)
                    if (!VEC && it.is_in && v[p][e] != v[p][e]) big = INFINITY;
                }
        };
        for (int s = 0; s < steps; ++s) {
            fetch(s);
            note(ia, va);
            if (tid < 16) note(ib, vb);
        }
        if (__syncthreads_or(big > kBf16Max)) {
            clear();
            strip(std::true_type{});
        }
    }
    // lane (q, j) holds rows 4 q + r (output channel), column j (input channel)
    if (!live) return;
    const long base = (long)blockIdx.x * Co * Ci * 9;
    const int ci = ci0 + cih * 16 + lj;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int co = co0 + coh * 16 + 4 * lq + r;
        if (co >= Co) continue;
        if (ci < Ci) {
            float v[9];
#pragma unroll
            for (int t = 0; t < 9; ++t) v[t] = sum_parts(acc[t][r], sml[t][r]);
            store_floats<9>(part + base + ((long)co * Ci + ci) * 9, v);
        }
        if (bias && lj == 0) gstore(partb + (long)blockIdx.x * Co + co, sum_parts(bm[r], bs[r]));
    }
}

// Rows per strip: 32, halved (down to 8) while a launch has fewer than 1024
// workgroups (four per CU).
int tr_wgrad_rows(int H, int W, int Ci, int Co, int nf)
{
    int rows = 32;
    auto groups = [&](int r) {
        return (long)nf * ((W + 31) / 32) * ((H + r - 1) / r) * ((Ci + 31) / 32) * ((Co + 31) / 32);
    };
    while (rows > 8 && groups(rows) < 1024) rows /= 2;
    return rows;
}

int tr_wgrad_strips(int H, int W, int Ci, int Co, int nf)
{
    const int r = tr_wgrad_rows(H, W, Ci, Co, nf);
    return nf * ((W + 31) / 32) * ((H + r - 1) / r);
}

hipError_t launch_wgrad_split(int H, int W, int Co, int ldg, int nf, const float *gm, long sgm, const float *in,
                              long sin, int Cf, const float *up, long sup, int Cu, float *part, float *partb,
                              hipStream_t s)
{
    const int Ci = Cu + Cf, rows = tr_wgrad_rows(H, W, Ci, Co, nf);
    if (Cu % 16 || ldg % 4 || (Cu > 0 && (H % 2 || W % 2))) return hipErrorInvalidValue;
    const int sx = (W + 31) / 32, sy = (H + rows - 1) / rows;
    const dim3 grid((unsigned)(nf * sx * sy), (unsigned)((Co + 31) / 32), (unsigned)((Ci + 31) / 32));
    if (Cf % 4 == 0)
        hipLaunchKernelGGL(tr_wgrad_split_kernel<true>, grid, dim3(256), 0, s, H, W, Co, ldg, rows, sx, sy, gm, sgm, in,
                           sin, Cf, up, sup, Cu, part, partb);
    else
        hipLaunchKernelGGL(tr_wgrad_split_kernel<false>, grid, dim3(256), 0, s, H, W, Co, ldg, rows, sx, sy, gm, sgm, in,
                           sin, Cf, up, sup, Cu, part, partb);
    return hipGetLastError();
}

}  // namespace wskp
