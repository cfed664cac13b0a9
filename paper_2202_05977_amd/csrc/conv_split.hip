// FP32 3x3 convolutions on the bf16 matrix cores: every fp32 operand is
// split into three bf16 parts, x = x0 + x1 + x2 (split_bf16; exact from 2^-110
// up), and a product is the sum of the six part products above 2^-25 of it:
//   x w = x0 w0 + (x1 w0 + x0 w1) + (x1 w1 + x2 w0 + x0 w2) + O(2^-25)
// Part products are exact in the MFMA, which accumulates in fp32.  x0 w0 goes
// into one accumulator and the five small terms into another; the two are
// added once at the end.  Against float64 the result is closer than that of
// v_mfma_f32_16x16x4f32 (random data, K = 32 .. 8192: error 1.1e-7 .. 5.8e-7
// against 1.0e-7 .. 1.6e-6): the main accumulator is rounded once per 16
// values of K, not once per 4, and the small terms' roundings are 2^-8 of
// its.  All six in one accumulator would be less exact than the fp32 form on
// data of one sign (the MFMA's sums round towards zero).
//
// Cost: 6 x 2 MFMAs of 32 cycles (v_mfma_f32_32x32x16_bf16) replace the 64 of
// v_mfma_f32_16x16x4f32 that 32 channels x 32 pixels x 32 values of K take at 32 cycles
// each: 2.7 times the rate (2.5 PFLOP/s / 6 against 157 TFLOP/s).
//
// A workgroup of 4 waves owns a tile of 4 HW x 32 output pixels and 32 output
// channels; a wave owns HW rows.  Per chunk of 16 input channels the halo is
// loaded as fp32 (one chunk ahead, in registers), split and written to LDS as
// three planes of bf16, with the chunk's weights (split when packed) beside
// it.  16 channels: at HW = 2 the stage is 59 KiB, so two workgroups fit a CU
// and one's staging hides behind the other's MFMAs; 32 would leave one.  The
// chunk is one k-step of the 32x32x16 form, and for one column offset dx a
// wave reads the fragments of its HW + 2 input rows once for up to three
// vertical taps: 75 bytes of LDS per clock and CU against the 128 it has.
//
// Measured, 1280x720 hd net: frame 1458 -> 945 us; dec0 (96 -> 32 channels)
// 456 -> 245 us = 208 TFLOP/s of fp32 work, 1248 of bf16 MFMAs; the card runs
// 32x32x16 MFMAs on random data from registers at 1830 (1.83 GHz: the clock
// gives way).
//
// Infinities and NaNs come out as in a plain fp32 sum (sum_parts), at no cost:
// the sums of an output with a NaN among its operands are as long as any.
#include "conv_device.h"

namespace wskp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32v4 __attribute__((ext_vector_type(4)));

constexpr int kSpCK = 16;                       // input channels per chunk
constexpr int kSpFrag = 1024;                   // bytes of one weight fragment (32 channels x 16)
constexpr int kSpWFrags = 9 * 3;                // fragments per chunk and 32 output channels

// Epilogues of the input gradients in training: what the gradient gm of the
// layer's input becomes is written at once, so it is itself never stored.
// Lane: pixel (y + r, x), channels co0 + 8 q + k.  Operands in the frame's
// descriptor: e[1] destination, u[0] activation whose ReLU masks it, e[2]
// second destination.
//   EPI_BWD_MASK  e[1] = (u[0] > 0) gm                        (the head's input)
//   EPI_BWD_CAT   channels below L.C1, the upsampled part of a decoder's input:
//                 e[1][y/2][x/2] = (u[0] > 0) (sum of the 2x2 block); the others,
//                 the skip: e[2] = gm (its first contribution)
//   EPI_BWD_POOL  the 2x2 mean's adjoint added to the finer map e[1] and its
//                 ReLU mask: e[1] = (u[0] > 0) (e[1] + gm / 4), 4 finer pixels
template <int EPI, int HW>
__device__ __forceinline__ void bwd_epilogue(const ConvLayer &L, const FrameDesc &fd, const f32x16 *acc, int co0,
                                             int y, int x, int Hl, int Wl)
{
    float *dst = static_cast<float *>(fd.e[1]);
    const float *act = static_cast<const float *>(fd.u[0]);
    auto mask = [](const gf32x4 &v, const gf32x4 &a) {
        return gf32x4{a[0] > 0.f ? v[0] : 0.f, a[1] > 0.f ? v[1] : 0.f, a[2] > 0.f ? v[2] : 0.f, a[3] > 0.f ? v[3] : 0.f};
    };
    auto at = [](auto *p, size_t i) { return reinterpret_cast<std::conditional_t<
        std::is_const_v<std::remove_pointer_t<decltype(p)>>, const gf32x4, gf32x4> *>(p + i); };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int co = co0 + 8 * q;
        const bool cin = co < L.Cout;
        if constexpr (EPI == EPI_BWD_CAT) {
            // (the channels of one q lie on one side: C1 is a multiple of 16)
            const int Cu = L.C1, Ce = L.Cout - Cu;
            if (co < Cu) {
                static_assert(EPI != EPI_BWD_CAT || HW == 2, "a 2x2 block in one wave");
                gf32x4 v;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float a = acc[0][4 * q + k], c = acc[HW - 1][4 * q + k];
                    v[k] = ((a + lane_xor1(a)) + c) + lane_xor1(c);
                }
                if ((x & 1) == 0 && y < Hl && x < Wl) {
                    const size_t i = ((size_t)(y >> 1) * (Wl >> 1) + (x >> 1)) * Cu + co;
                    gstore(at(dst, i), mask(v, gload(at(act, i))));
                }
            } else if (cin) {
                float *ge = static_cast<float *>(fd.e[2]);
#pragma unroll
                for (int r = 0; r < HW; ++r)
                    if (y + r < Hl && x < Wl)
                        gstore(at(ge, ((size_t)(y + r) * Wl + x) * Ce + (co - Cu)),
                               gf32x4{acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]});
            }
        } else {
#pragma unroll
            for (int r = 0; r < HW; ++r) {
                if (!cin || y + r >= Hl || x >= Wl) continue;
                const gf32x4 v = {acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]};
                if constexpr (EPI == EPI_BWD_MASK) {
                    const size_t i = ((size_t)(y + r) * Wl + x) * L.Cout + co;
                    gstore(at(dst, i), mask(v, gload(at(act, i))));
                } else {
                    gf32x4 o[4], a[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const size_t i = ((size_t)(2 * (y + r) + (k >> 1)) * (2 * Wl) + 2 * x + (k & 1)) * L.Cout + co;
                        o[k] = gload(at(const_cast<const float *>(dst), i));
                        a[k] = gload(at(act, i));
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const size_t i = ((size_t)(2 * (y + r) + (k >> 1)) * (2 * Wl) + 2 * x + (k & 1)) * L.Cout + co;
                        gstore(at(dst, i), mask(o[k] + 0.25f * v, a[k]));
                    }
                }
            }
        }
    }
}

template <int MODE, int EPI, int HW>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_split_kernel(ConvLayer L, FrameArg fa)
{
    constexpr int TH = 4 * HW, HP = TH + 2, WP = kConvTW + 2, NPIX = HP * WP;
    constexpr int PART = NPIX * 32;                        // bytes of one part's plane: 16 bf16 per pixel
    constexpr int A_BYTES = 3 * PART, W_BYTES = kSpWFrags * kSpFrag;
    // staging items: a pixel's run of 8 channels (network input: a pixel)
    constexpr bool PACK = MODE == CONV_PACK;
    constexpr int NG = PACK ? 1 : 2, NI = NPIX * NG, IT = (NI + kThreads - 1) / kThreads;
    constexpr int WSLOTS = W_BYTES / 16, WIT = (WSLOTS + kThreads - 1) / kThreads;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[A_BYTES + W_BYTES];

    int f, g, x0, y0, Hl, Wl;
    if (!conv_locate<TH>(L, fa, f, g, x0, y0, Hl, Wl)) return;
    const FrameDesc &fd = frame_at(fa, f);
    const float *s0 = reinterpret_cast<const float *>(conv_src0(L, fd));
    const float *s1 = reinterpret_cast<const float *>(fd.e[L.src1_idx]);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 31, lh = lane >> 5;
    const int nch = L.Cin_pad / kSpCK;

    // ---- staging: element offsets of this thread's items, and where they go.
    // LDS holds 32 bytes per pixel and part; a pixel's two 16-byte groups are
    // swapped where bit 2 of its column is set, so that the 8 consecutive
    // pixels a fragment read takes per cycle hit distinct banks.
    // Loads are buffer loads: items outside the image take an offset beyond the
    // buffer and read zeros (the conv's zero padding).
    constexpr unsigned kOut = 0x7ffffff0u;   // maps stay below 2 GiB - 64 KiB
    const unsigned px = (unsigned)Hl * Wl, cp = (unsigned)L.C0 * 4u;
    unsigned n0 = px * cp;                   // bytes of source 0
    if (MODE == CONV_CAT) n0 = (unsigned)(Hl >> 1) * (Wl >> 1) * cp;
    if (MODE == CONV_POOL) n0 = 4u * px * cp;
    const rsrc_t r0 = make_rsrc(s0, PACK ? 0u : n0);
    const rsrc_t r1 = make_rsrc(s1, MODE == CONV_CAT ? px * (unsigned)L.C1 * 4u : 0u);
    const rsrc_t rr = make_rsrc(fd.r, px * 12u), ra = make_rsrc(fd.a, px * 12u), rn = make_rsrc(fd.n, px * 12u),
                 rd = make_rsrc(fd.d, px * 4u);
    unsigned off0[IT], off1[MODE == CONV_CAT ? IT : 1];
    int dst[IT];
    unsigned live = 0;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int it = tid + k * kThreads;
        const int p = it / NG, cg = it - p * NG;
        const int ly = p / WP, lx = p - ly * WP;
        const int gy = y0 - 1 + ly, gx = x0 - 1 + lx;
        const bool ok = it < NI && gy >= 0 && gy < Hl && gx >= 0 && gx < Wl;
        live |= ok ? 1u << k : 0u;
        dst[k] = p * 32 + ((cg ^ ((lx >> 2) & 1)) << 4);
        if constexpr (PACK) off0[k] = ok ? (unsigned)(gy * Wl + gx) : kOut / 12u;
        else if constexpr (MODE == CONV_PLAIN) off0[k] = ok ? (unsigned)(gy * Wl + gx) * cp + cg * 32 : kOut;
        else if constexpr (MODE == CONV_CAT) {
            off0[k] = ok ? (unsigned)((gy >> 1) * (Wl >> 1) + (gx >> 1)) * cp + cg * 32 : kOut;
            off1[k] = ok ? (unsigned)(gy * Wl + gx) * ((unsigned)L.C1 * 4u) + cg * 32 : kOut;
        } else off0[k] = ok ? (unsigned)(2 * gy * (2 * Wl) + 2 * gx) * cp + cg * 32 : kOut;
    }
    const unsigned char *wsrc = static_cast<const unsigned char *>(L.w) + (size_t)g * nch * W_BYTES;
    const rsrc_t rw = make_rsrc(wsrc, (unsigned)(nch * W_BYTES));

    auto load4 = [](rsrc_t r, unsigned voff, int soff) {
        return __builtin_bit_cast(gf32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0));
    };
    float in[IT][PACK ? 10 : 8];
    u32v4 w[WIT];
    auto fetch = [&](int cc) {
        const int c0 = cc * kSpCK;
        const bool up = MODE != CONV_CAT || c0 < L.C0;
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            if constexpr (PACK) {
                const auto vr = __builtin_amdgcn_raw_buffer_load_b96(rr, (int)(off0[k] * 12u), 0, 0);
                const auto va = __builtin_amdgcn_raw_buffer_load_b96(ra, (int)(off0[k] * 12u), 0, 0);
                const auto vn = __builtin_amdgcn_raw_buffer_load_b96(rn, (int)(off0[k] * 12u), 0, 0);
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    in[k][e] = __uint_as_float(vr[e]);
                    in[k][3 + e] = __uint_as_float(va[e]);
                    in[k][6 + e] = __uint_as_float(vn[e]);
                }
                in[k][9] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rd, (int)(off0[k] * 4u), 0, 0));
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    gf32x4 v;
                    if constexpr (MODE == CONV_POOL) {
                        const int rs = 2 * Wl * (int)cp, at = (c0 + 4 * q) * 4;
                        const gf32x4 a0 = load4(r0, off0[k], at), a1 = load4(r0, off0[k], at + (int)cp);
                        const gf32x4 a2 = load4(r0, off0[k], at + rs), a3 = load4(r0, off0[k], at + rs + (int)cp);
                        v = 0.25f * (a0 + a1 + a2 + a3);
                    } else if (up) {
                        v = load4(r0, off0[k], (c0 + 4 * q) * 4);
                    } else {
                        v = load4(r1, off1[MODE == CONV_CAT ? k : 0], (c0 - L.C0 + 4 * q) * 4);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) in[k][4 * q + e] = v[e];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < WIT; ++k)
            w[k] = __builtin_bit_cast(u32v4, __builtin_amdgcn_raw_buffer_load_b128(
                                                 rw, (tid + k * kThreads) * 16, cc * W_BYTES, 0));
    };
    auto commit = [&]() {
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            if (tid + k * kThreads >= NI) continue;
            if constexpr (PACK) {
                float x[16];
                pack_transform(L, in[k]);
#pragma unroll
                for (int e = 0; e < 16; ++e) x[e] = e < 10 && ((live >> k) & 1u) ? in[k][e < 10 ? e : 0] : 0.f;
#pragma unroll
                for (int cg = 0; cg < 2; ++cg) {
                    unsigned p[4][3];
                    split_bf16_run(x + cg * 8, p);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        *reinterpret_cast<uint4 *>(&smem[q * PART + (dst[k] ^ (cg << 4))]) =
                            make_uint4(p[0][q], p[1][q], p[2][q], p[3][q]);
                }
            } else {
                unsigned p[4][3];
                split_bf16_run(in[k], p);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint4 *>(&smem[q * PART + dst[k]]) =
                        make_uint4(p[0][q], p[1][q], p[2][q], p[3][q]);
            }
        }
#pragma unroll
        for (int k = 0; k < WIT; ++k)
            if (tid + k * kThreads < WSLOTS)
                *reinterpret_cast<u32v4 *>(&smem[A_BYTES + (tid + k * kThreads) * 16]) = w[k];
    };

    f32x16 acc[HW], sml[HW];
#pragma unroll
    for (int r = 0; r < HW; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[r][i] = sml[r][i] = 0.f;

    auto frag = [&](int at) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32v4 *>(&smem[at]));
    };
    // per column offset: this lane's pixel of row 0 of its wave, with its group's place
    int abase[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
        abase[dx] = (wave * HW * WP + lj + dx) * 32 + ((lh ^ (((lj + dx) >> 2) & 1)) << 4);
    // Taps in the order dx, dy.  The fragments of the next tap (its weights and
    // the input rows it adds) are requested before the MFMAs of this one, so
    // that these (12 x 32 cycles) cover the LDS latency; left to itself the
    // compiler reads each fragment just before its first use.
    auto compute = [&]() {
        bf16x8 x[3][HW + 2][3], k[9][3];
        auto load_row = [&](int dx, int rr) {
#pragma unroll
            for (int q = 0; q < 3; ++q) x[dx][rr][q] = frag(abase[dx] + q * PART + rr * WP * 32);
        };
        auto load_w = [&](int dx, int dy) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
                k[dx * 3 + dy][q] = frag(A_BYTES + ((dy * 3 + dx) * 3 + q) * kSpFrag + lane * 16);
        };
#pragma unroll
        for (int rr = 0; rr < HW; ++rr) load_row(0, rr);
        load_w(0, 0);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int dx = t / 3, dy = t % 3;
            if (dy < 2) {
                load_row(dx, HW + dy);
                load_w(dx, dy + 1);
            } else if (dx < 2) {
#pragma unroll
                for (int rr = 0; rr < HW; ++rr) load_row(dx + 1, rr);
                load_w(dx + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            auto mm = [&](int kq, int xq, f32x16 *c) {
#pragma unroll
                for (int r = 0; r < HW; ++r)
                    c[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k[t][kq], x[dx][r + dy][xq], c[r], 0, 0, 0);
            };
            mm(2, 0, sml);
            mm(0, 0, acc);
            mm(0, 2, sml);
            mm(1, 1, sml);
            mm(1, 0, sml);
            mm(0, 1, sml);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    fetch(0);
    for (int cc = 0; cc < nch; ++cc) {
        if (cc) lds_sync();   // every wave has read the chunk before
        commit();
        lds_sync();
        if (cc + 1 < nch) fetch(cc + 1);
        compute();
    }

    // ---- epilogue: lane (j, h) holds pixel j of its rows, channels
    // 8 q + 4 h .. + 3 for q = 0..3
    const int co0 = g * 32 + 4 * lh;
#pragma unroll
    for (int r = 0; r < HW; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[r][i] = sum_parts(acc[r][i], sml[r][i]);
    if constexpr (EPI == EPI_BWD_MASK || EPI == EPI_BWD_CAT || EPI == EPI_BWD_POOL) {
        bwd_epilogue<EPI, HW>(L, fd, acc, co0, y0 + wave * HW, x0 + lj, Hl, Wl);
        return;
    }
    float bias[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int co = co0 + 8 * (i >> 2) + (i & 3);
        bias[i] = co < L.Cout ? gload(L.bias + co) : 0.f;
    }
    float *out = conv_dst<float>(L, fd);
    const size_t P = (size_t)Hl * Wl;
#pragma unroll
    for (int r = 0; r < HW; ++r) {
        const int y = y0 + wave * HW + r, x = x0 + lj;
        if (y >= Hl || x >= Wl) continue;
        const size_t pix = (size_t)y * Wl + x;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int co = co0 + 8 * q;
            if (co >= L.Cout) continue;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = epilogue<EPI>(acc[r][4 * q + k] + bias[4 * q + k], co + k, L.M);
            if constexpr (EPI == EPI_HEAD_SOFTPLUS || EPI == EPI_HEAD_EXP) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (co + k < L.Cout) gstore(out + (size_t)(co + k) * P + pix, v[k]);
            } else {
                // Cout is a multiple of 16
                gstore(reinterpret_cast<gf32x4 *>(out + pix * L.Cout + co), gf32x4{v[0], v[1], v[2], v[3]});
            }
        }
    }
}

// ---- weights ------------------------------------------------------------------
size_t conv_split_weight_bytes(int Cin, int Cout)
{
    return (size_t)((Cout + 31) / 32) * ((Cin + kSpCK - 1) / kSpCK) * kSpWFrags * kSpFrag;
}

// Weight packing, all layers in one launch.  Packed split weights of a conv
// Ci -> Co: fragments [group of 32 output channels][chunk][tap][part], in each
// lane (h, j)'s 8 values for output channel j of the group and input channels
// 8 h .. 8 h + 7 of the chunk; zero beyond Ci or Co.  PACK_SPLIT: w is
// [Co][Ci][3][3].  PACK_SPLIT_DGRAD: the conv that maps the gradient of w's
// output to its input's (taps flipped, channel axes swapped), w [Ci][Co][3][3].
// PACK_NATIVE: the layout of the v_mfma_f32_16x16x4f32 kernel, [chunk of CK]
// [tap][c][Cout_pad] floats, and the Co biases after w to `bias`.
__global__ __launch_bounds__(kThreads) void conv_pack_kernel(PackJobs jobs)
{
    int b = blockIdx.x, j = 0;
    while (j + 1 < jobs.n && b >= jobs.j[j + 1].block0) ++j;
    const PackJob &p = jobs.j[j];
    const int i = (b - p.block0) * kThreads + threadIdx.x;
    if (p.kind == PACK_NATIVE) {
        const int n = p.nch * 9 * p.CK * p.Cout_pad;
        if (i < n) {
            const int co = i % p.Cout_pad, c = i / p.Cout_pad % p.CK, t = i / (p.Cout_pad * p.CK) % 9;
            const int ci = i / (p.Cout_pad * p.CK * 9) * p.CK + c;
            gstore(static_cast<float *>(p.out) + i,
                   co < p.Co && ci < p.Ci ? gload(p.w + ((size_t)co * p.Ci + ci) * 9 + t) : 0.f);
        } else if (i < n + p.Co) {
            gstore(p.bias + (i - n), gload(p.w + (size_t)p.Co * p.Ci * 9 + (i - n)));
        }
        return;
    }
    if (i >= p.groups * p.nch * 9 * 512) return;            // (group, chunk, tap, lane, e)
    const int e = i & 7, lane = (i >> 3) & 63, t = i / 512 % 9, cc = i / (512 * 9) % p.nch, gr = i / (512 * 9 * p.nch);
    const int co = gr * 32 + (lane & 31), ci = cc * kSpCK + (lane >> 5) * 8 + e;
    float v = 0.f;
    if (co < p.Co && ci < p.Ci)
        v = gload(p.kind == PACK_SPLIT_DGRAD ? p.w + ((size_t)ci * p.Co + co) * 9 + (8 - t)
                                             : p.w + ((size_t)co * p.Ci + ci) * 9 + t);
    unsigned short *o = static_cast<unsigned short *>(p.out) + ((size_t)((gr * p.nch + cc) * 9 + t) * 3) * 512 + lane * 8 + e;
    unsigned parts[3];
    split_bf16<true>(v, 0.f, parts);
#pragma unroll
    for (int q = 0; q < 3; ++q) gstore(o + q * 512, (unsigned short)parts[q]);
}

void PackJobs::add_split(int Ci, int Co, bool dgrad, const float *w, void *out)
{
    PackJob &p = j[n++];
    p = PackJob{};
    p.kind = dgrad ? PACK_SPLIT_DGRAD : PACK_SPLIT;
    p.Ci = Ci;
    p.Co = Co;
    p.nch = (Ci + kSpCK - 1) / kSpCK;
    p.groups = (Co + 31) / 32;
    p.w = w;
    p.out = out;
    p.block0 = blocks;
    blocks += (p.groups * p.nch * 9 * 512 + kThreads - 1) / kThreads;
}

void PackJobs::add_native(int Ci, int Co, int CK, int nch, int Cout_pad, const float *w, float *out, float *bias)
{
    PackJob &p = j[n++];
    p = PackJob{};
    p.kind = PACK_NATIVE;
    p.Ci = Ci;
    p.Co = Co;
    p.CK = CK;
    p.nch = nch;
    p.Cout_pad = Cout_pad;
    p.w = w;
    p.out = out;
    p.bias = bias;
    p.block0 = blocks;
    blocks += (nch * 9 * CK * Cout_pad + Co + kThreads - 1) / kThreads;
}

hipError_t launch_conv_pack(const PackJobs &jobs, hipStream_t s)
{
    if (jobs.n == 0) return hipSuccess;
    hipLaunchKernelGGL(conv_pack_kernel, dim3(jobs.blocks), dim3(kThreads), 0, s, jobs);
    return hipGetLastError();
}

// ---- dispatch -------------------------------------------------------------------
void conv_split_layer(ConvLayer &L, int Cin)
{
    L.CK = kSpCK;
    L.Cin_pad = (Cin + kSpCK - 1) / kSpCK * kSpCK;
    L.NB = 2;
    L.groups = (L.Cout + 31) / 32;
    L.Cout_pad = L.groups * 32;
    L.th = 8;
}

template <int MODE, int EPI>
static hipError_t launch_split_inst(const ConvLayer &L, const FrameArg &fa, int blocks, hipStream_t s)
{
    if constexpr (EPI == EPI_BWD_CAT) {
        if (L.th != 8) return hipErrorInvalidValue;
    } else if (L.th == 4) {
        hipLaunchKernelGGL((conv3x3_split_kernel<MODE, EPI, 1>), dim3(blocks), dim3(kThreads), 0, s, L, fa);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((conv3x3_split_kernel<MODE, EPI, 2>), dim3(blocks), dim3(kThreads), 0, s, L, fa);
    return hipGetLastError();
}

hipError_t launch_conv_split(const ConvLayer &L, int mode, int epi, const FrameArg &fa, int blocks, hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    if (L.ks != 3 || (L.th != 4 && L.th != 8)) return hipErrorInvalidValue;
    switch (mode) {
    case CONV_PACK: return launch_split_inst<CONV_PACK, EPI_RELU>(L, fa, blocks, s);
    case CONV_POOL: return launch_split_inst<CONV_POOL, EPI_RELU>(L, fa, blocks, s);
    case CONV_CAT: return launch_split_inst<CONV_CAT, EPI_RELU>(L, fa, blocks, s);
    case CONV_PLAIN:
        if (epi == EPI_BWD_MASK) return launch_split_inst<CONV_PLAIN, EPI_BWD_MASK>(L, fa, blocks, s);
        if (epi == EPI_BWD_CAT) return launch_split_inst<CONV_PLAIN, EPI_BWD_CAT>(L, fa, blocks, s);
        if (epi == EPI_BWD_POOL) return launch_split_inst<CONV_PLAIN, EPI_BWD_POOL>(L, fa, blocks, s);
        if (epi == EPI_HEAD_EXP) return launch_split_inst<CONV_PLAIN, EPI_HEAD_EXP>(L, fa, blocks, s);
        if (epi == EPI_HEAD_SOFTPLUS) return launch_split_inst<CONV_PLAIN, EPI_HEAD_SOFTPLUS>(L, fa, blocks, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

}  // namespace wskp
