// bf16 convolutions (3x3, or 5x5 for merged RepVGG blocks) of layers whose
// input channels come in chunks of 32 and whose output channels are a
// multiple of 32: implicit GEMM with v_mfma_f32_32x32x16_bf16.
//
// A workgroup of 4 waves owns a tile of 4 R x 32 output pixels and 32 output
// channels; a wave owns R rows, each one 32-pixel MFMA column block.  Per
// chunk the halo and the weights go from memory straight into LDS
// (buffer_load_dwordx4 ... lds); for one column offset dx a wave reads the
// fragments of its R + KS - 1 input rows once and uses each for up to KS
// vertical taps.
//
// Why this shape.  v_mfma_f32_32x32x16_bf16 keeps the matrix pipe full from one
// wave (32 cycles each; v_mfma_f32_16x16x32_bf16 measured 31 cycles instead of
// 16 from one wave, 19.5 from two or more), and two of them over the halves of
// 32 values of K give bitwise the sum of one 16x16x32.  LDS reads per MFMA fall
// with R: 3x3, 1.17 KiB at R = 2, 0.89 at R = 3 (a CU reads 4 KiB in the 32
// cycles its four SIMDs take for one MFMA each).
//
// What bounds it: memory, LDS and the matrix cores take about the same time
// each and overlap in part.  dec0 of 6.9 Mpixels (96 -> 32 channels), 376 us:
// 1.1 GB at the 5.1 TB/s of a large copy 216, MFMAs at the clock they leave
// (1830 TFLOP/s) 209, LDS reads about 200; without its stores it takes 306,
// without staging 295, without MFMAs 331.
// Tried and slower: the next chunk prefetched into registers (dec0 at 720p 65 us
// against 56), persistent workgroups that load the next tile under the
// epilogue (59), 16-row tiles (60).
//
// Measured against 16x16x32 MFMAs with per-chunk address arithmetic and
// 32-byte stores, both in turn on one card, frame times, bitwise the same output:
// 5x5 net at 720p 474 -> 451 us, the six-kernel net at 664x376 123 -> 114; the 3x3
// net at 720p 250 -> 249 and a batch of 360p..1440p 1600 -> 1584, hardly more than
// the runs differ: there the card's power, not the kernel's issue, sets the
// decoders' pace (a card that holds its clock: 243 -> 234).
//
// LDS images.  Halo: 64 bytes a pixel, its four 16-byte channel groups at
// position g ^ ((column >> 1) & 3), so that the 8 consecutive pixels that one
// cycle of a fragment read takes hit distinct banks; the order depends on the
// column alone, so a lane needs one address per dx and half of K and every
// row is an immediate offset.  Weights: fragments in lane order, 1 KiB each.
#include "conv_device.h"

namespace wskp {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kDirCK = 32;
// Stage: 3x3, 31, 40 and 48 KiB for R = 1, 2, 3 (five, four, three workgroups
// per CU); 5x5, 68 and 77 KiB for R = 1, 2 (two).
constexpr int dir_halo_ins(int KS, int R) { return ((4 * R + KS - 1) * (kConvTW + KS - 1) * 4 + 63) / 64; }
constexpr int dir_stage_bytes(int KS, int R) { return (dir_halo_ins(KS, R) + KS * KS * 2) * 1024; }
constexpr int dir_min_wg(int KS, int R)
{
    return 163840 / dir_stage_bytes(KS, R) < 4 ? 163840 / dir_stage_bytes(KS, R) : 4;
}

constexpr unsigned kDirOut = 0x7ffffff0u;   // beyond every buffer: such loads write zeros

template <int MODE, int KS, int R, bool POOL>
__global__ __launch_bounds__(kThreads, dir_min_wg(KS, R)) void conv_bf16_kernel(ConvLayer L, FrameArg fa)
{
    constexpr int TH = 4 * R, HP = TH + KS - 1, WP = kConvTW + KS - 1, NPIX = HP * WP;
    constexpr int A_INS = dir_halo_ins(KS, R), W_INS = KS * KS * 2;
    constexpr int AW = (A_INS + 3) / 4, WW = (W_INS + 3) / 4;   // load instructions per wave
    constexpr int A_BYTES = A_INS * 1024;
    static_assert(!POOL || R % 2 == 0, "2x2 means need whole row pairs per wave");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[dir_stage_bytes(KS, R)];

    int f, g, x0, y0, Hl, Wl;
    if (!conv_locate<TH>(L, fa, f, g, x0, y0, Hl, Wl)) return;
    const FrameDesc &fd = frame_at(fa, f);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 31, lh = lane >> 5;

    const void *s0 = conv_src0(L, fd);
    const void *s1 = fd.e[L.src1_idx];
    const int H0 = MODE == CONV_CAT ? Hl >> 1 : Hl, W0 = MODE == CONV_CAT ? Wl >> 1 : Wl;
    const rsrc_t r0 = make_rsrc(s0, (unsigned)((size_t)H0 * W0 * L.C0 * 2));
    const rsrc_t r1 = make_rsrc(s1, MODE == CONV_CAT ? (unsigned)((size_t)Hl * Wl * L.C1 * 2) : 0u);
    const int nch = L.Cin_pad / kDirCK;
    const rsrc_t rw = make_rsrc(static_cast<const unsigned char *>(L.w) + (size_t)g * nch * (W_INS * 1024),
                                (unsigned)(nch * (W_INS * 1024)));

    // Byte offsets (chunk 0) of this lane's halo slots in source 0 and source
    // 1; the lane's k-th slot is slot0 + 256 k, halo pixel p0 + 64 k.  Pixels
    // outside the image, and slots past the halo, get kDirOut.  Row and pixel
    // pitches are below 2^24: 24-bit multiplies.
    const unsigned cp0 = (unsigned)L.C0 * 2u, rp0 = (unsigned)W0 * cp0;
    const unsigned cp1 = (unsigned)L.C1 * 2u, rp1 = (unsigned)Wl * cp1;
    const int p0 = wave * 16 + (lane >> 2);
    constexpr int SY = 64 / WP, SX = 64 - SY * WP;
    int ly = p0 / WP, lx = p0 - ly * WP;
    unsigned oa0[AW], oa1[MODE == CONV_CAT ? AW : 1];
#pragma unroll
    for (int k = 0; k < AW; ++k) {
        const int gy = y0 - KS / 2 + ly, gx = x0 - KS / 2 + lx;
        const bool in = p0 + 64 * k < NPIX && (unsigned)gy < (unsigned)Hl && (unsigned)gx < (unsigned)Wl;
        const unsigned go = (unsigned)(((lane & 3) ^ ((lx >> 1) & 3)) * 16);
        if constexpr (MODE == CONV_CAT) {
            oa0[k] = in ? __umul24((unsigned)gy >> 1, rp0) + __umul24((unsigned)gx >> 1, cp0) + go : kDirOut;
            oa1[k] = in ? __umul24((unsigned)gy, rp1) + __umul24((unsigned)gx, cp1) + go : kDirOut;
        } else {
            oa0[k] = in ? __umul24((unsigned)gy, rp0) + __umul24((unsigned)gx, cp0) + go : kDirOut;
        }
        lx += SX;
        ly += SY;
        if (lx >= WP) {
            lx -= WP;
            ++ly;
        }
    }
    auto load_lds = [&](rsrc_t r, int ins, unsigned voff, int soff) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, (__attribute__((address_space(3))) void *)(smem + ins * 1024), 16, (int)voff, soff, 0, 0);
    };
    // issues chunk cc's loads: instruction j of the halo fills slots 64 j ..,
    // instruction j of the weights is fragment j
    auto issue = [&](int cc) {
        const int c0 = cc * kDirCK;
        const bool up = MODE != CONV_CAT || c0 < L.C0;
        const int da = (up ? c0 : c0 - L.C0) * 2;
#pragma unroll
        for (int k = 0; k < AW; ++k) {
            const int ins = wave + 4 * k;
            if (4 * k + 3 < A_INS || ins < A_INS) {
                if (up) load_lds(r0, ins, oa0[k], da);
                else load_lds(r1, ins, oa1[MODE == CONV_CAT ? k : 0], da);
            }
        }
#pragma unroll
        for (int k = 0; k < WW; ++k) {
            const int ins = wave + 4 * k;
            if (4 * k + 3 < W_INS || ins < W_INS)
                load_lds(rw, A_INS + ins, (unsigned)(lane * 16), (cc * W_INS + ins) * 1024);
        }
    };

    f32x16 acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[r][i] = 0.f;

    // per column offset: this lane's pixel in its wave's first halo row, first
    // half of K; the second half is at the address ^ 32
    int ab[KS];
#pragma unroll
    for (int dx = 0; dx < KS; ++dx)
        ab[dx] = (wave * R * WP + lj + dx) * 64 + ((lh ^ (((lj + dx) >> 1) & 3)) << 4);
    auto frag = [&](int at) { return *reinterpret_cast<const bf16x8 *>(&smem[at]); };
    // One chunk.  Taps in the order dx, dy; the next tap's fragments (its
    // weights and the input rows it adds) are requested before this one's
    // MFMAs.  Once the last tap's have arrived the stage is free: the next
    // chunk's loads are issued under the last MFMAs.
    auto compute = [&](int cc) {
        constexpr int T = KS * KS;
        bf16x8 x[KS][R + KS - 1][2], w[T][2];
        auto load_row = [&](int dx, int rr) {
#pragma unroll
            for (int h = 0; h < 2; ++h) x[dx][rr][h] = frag((ab[dx] ^ (h * 32)) + rr * WP * 64);
        };
        auto load_w = [&](int t) {   // t counts in the order dx, dy
#pragma unroll
            for (int h = 0; h < 2; ++h)
                w[t][h] = frag(A_BYTES + ((t % KS * KS + t / KS) * 2 + h) * 1024 + lane * 16);
        };
#pragma unroll
        for (int rr = 0; rr < R; ++rr) load_row(0, rr);
        load_w(0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int dx = t / KS, dy = t % KS;
            if (t + 1 < T) {
                if (dy + 1 < KS) load_row(dx, R + dy);
                else
#pragma unroll
                    for (int rr = 0; rr < R; ++rr) load_row(dx + 1, rr);
                load_w(t + 1);
            } else {
                wait_lds();
                lds_barrier();
                if (cc + 1 < nch) issue(cc + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[t][h], x[dx][r + dy][h], acc[r], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    issue(0);
    for (int cc = 0; cc < nch; ++cc) {
        wait_vmem<0>();
        lds_barrier();
        compute(cc);
    }

    // ---- epilogue: lane (j, h) holds pixel j of its rows, channels
    // 8 q + 4 h .. + 3 for q = 0..3.  v_permlane32_swap exchanges the upper
    // half of block q with the lower half of block q + 1, after which each
    // lane holds 8 consecutive channels of block q + h.  The wave passes them
    // through its own part of the stage (no longer read: see the last barrier)
    // and stores 4 lanes to a pixel, 64 bytes each, whole lines for 16 pixels:
    // straight from the lanes above a store would cover 32 bytes a pixel.
    float bias[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) bias[i] = gload(L.bias + g * 32 + 8 * (i >> 2) + 4 * lh + (i & 3));
    unsigned short *dst = conv_dst<unsigned short>(L, fd) + g * 32 + (lane & 3) * 8;
    unsigned short *pdst = POOL ? reinterpret_cast<unsigned short *>(fd.p[L.pool_idx]) + g * 32 + (lane & 3) * 8 : nullptr;
    float pe[POOL ? 16 : 1];   // column-pair sums of the even row
    static_assert(4 * R * 3072 <= dir_stage_bytes(KS, R), "rows and means of every wave fit the stage");
    const int tr = wave * R * 3072;                    // a row: 2 KiB of pixels, 1 KiB of means
    // 16-byte group c of pixel p at group c ^ ((p >> 1) & 3): the 8 lanes of a
    // cycle hit distinct banks writing (8 pixels) and reading (2 pixels x 4)
    auto put = [&](int at, int p, int q, const uint2 &a, const uint2 &b, bool on) {
        const auto sx = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
        const auto sy = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
        if (on)
            *reinterpret_cast<gu32x4 *>(&smem[at + p * 64 + (((q + lh) ^ ((p >> 1) & 3)) << 4)]) =
                gu32x4{sx[0], sy[0], sx[1], sy[1]};
    };
    auto get = [&](int at, int p) {
        return *reinterpret_cast<const gu32x4 *>(&smem[at + p * 64 + (((lane & 3) ^ ((p >> 1) & 3)) << 4)]);
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint2 qs[4], pm[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = fmaxf(acc[r][4 * q + k] + bias[4 * q + k], 0.f);
            qs[q] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
            if constexpr (POOL) {
                const float s[4] = {__uint_as_float(qs[q].x << 16), __uint_as_float(qs[q].x & 0xffff0000u),
                                    __uint_as_float(qs[q].y << 16), __uint_as_float(qs[q].y & 0xffff0000u)};
                float m[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (r % 2 == 0) pe[4 * q + k] = s[k] + lane_xor1(s[k]);
                    else m[k] = 0.25f * ((pe[4 * q + k] + s[k]) + lane_xor1(s[k]));
                }
                if (r % 2) pm[q] = make_uint2(pack2(m[0], m[1]), pack2(m[2], m[3]));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            put(tr + r * 3072, lj, q, qs[q], qs[q + 1], true);
            // the mean is the even lane's, which adds its pair's columns in order
            // (the odd lane's sum of the odd row starts at the other column and
            // may round differently)
            if (POOL && r % 2) put(tr + r * 3072 + 2048, lj >> 1, q, pm[q], pm[q + 1], lj % 2 == 0);
        }
    }
    wait_lds();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + wave * R + r;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int px = k * 16 + (lane >> 2), x = x0 + px;
            const gu32x4 v = get(tr + r * 3072, px);
            if (y < Hl && x < Wl) gstore(reinterpret_cast<gu32x4 *>(dst + ((size_t)y * Wl + x) * L.Cout), v);
        }
        if (POOL && r % 2) {
            const int X = (x0 >> 1) + (lane >> 2), Y = y >> 1;
            const gu32x4 v = get(tr + r * 3072 + 2048, lane >> 2);
            if (Y < (Hl >> 1) && X < (Wl >> 1))
                gstore(reinterpret_cast<gu32x4 *>(pdst + ((size_t)Y * (Wl >> 1) + X) * L.Cout), v);
        }
    }
}

// Tile rows for a launch.
// 12 (3x3): fewer LDS bytes per MFMA and fewer weight bytes staged per pixel
// than 8, but three workgroups per CU instead of four, so it needs several
// rounds of the 768 that fit: a batch of 360p + 720p + 1080p + 1440p, dec0
// (18000 tiles) 376 us against 391, dec1 (9000) 275 against 294, dec2 (3405)
// 133 against 135; one 720p frame, dec0 (2400) 58 either way, dec2 (450) 29
// against 28.
// 4: where 8-row tiles are fewer than the 512 workgroups that put two on every
// CU (720p, level 3: 480 tiles 9.3 us, 240 tiles 9.9).  A layer that passes on
// 2x2 means keeps 8: it needs whole row pairs in a wave.
int conv_bf16_rows(const ConvLayer &L, int n, const int *H, const int *W)
{
    ConvLayer c = L;
    c.th = 12;
    if (L.ks == 3 && L.pool_idx < 0 && conv_grid(c, n, H, W) >= 3072) return 12;
    c.th = 8;
    return L.pool_idx >= 0 || conv_grid(c, n, H, W) >= 512 ? 8 : 4;
}

hipError_t launch_conv_bf16(const ConvLayer &L, int mode, const FrameArg &fa, int blocks, hipStream_t s)
{
#define WSKP_LAUNCH(MODE, K, R, POOL)                                                                               \
    if (L.ks == K && L.th == 4 * R && mode == MODE && (L.pool_idx >= 0) == POOL) {                                  \
        hipLaunchKernelGGL((conv_bf16_kernel<MODE, K, R, POOL>), dim3(blocks), dim3(kThreads), 0, s, L, fa);        \
        return hipGetLastError();                                                                                   \
    }
#define WSKP_KS(K)                                                                                                  \
    WSKP_LAUNCH(CONV_PLAIN, K, 2, true) WSKP_LAUNCH(CONV_PLAIN, K, 2, false) WSKP_LAUNCH(CONV_PLAIN, K, 1, false)   \
    WSKP_LAUNCH(CONV_CAT, K, 2, false) WSKP_LAUNCH(CONV_CAT, K, 1, false)
    WSKP_KS(3) WSKP_KS(5) WSKP_LAUNCH(CONV_PLAIN, 3, 3, false) WSKP_LAUNCH(CONV_CAT, 3, 3, false)
#undef WSKP_KS
#undef WSKP_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace wskp
