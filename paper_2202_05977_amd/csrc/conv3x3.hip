// Convolutions of the prediction network (Sec. 4.1, Eq. 2) as implicit
// GEMMs on the gfx950 matrix cores: 3x3, or 5x5 for a net whose convs are
// merged RepVGG blocks (Sec. 4.1, prediction phase).
//
// GEMM view of one layer: output pixels x output channels, reduction K =
// KS*KS taps x C_in (the MFMAs take the weights as their first operand, so
// each lane ends with 4 consecutive channels of one pixel, which the
// epilogue stores directly).  A workgroup (4 wave64s) owns a tile of
// TH x 32 output pixels and 16*NB output channels.  The reduction runs over
// chunks of CK input channels: the (TH+KS-1) x (32+KS-1) input halo of the
// chunk and the matching KS*KS*CK x 16*NB weight slice are staged in LDS,
// then every wave issues MFMAs over the taps.  The operation that produces the layer's
// input is fused into the staging step, so that input never exists in
// memory:
//   CONV_PACK   network input (Sec. 5.1): gamma-tonemapped radiance, albedo,
//               (normal+1)/2 and clamped scaled depth, from the raw buffers
//   CONV_POOL   2x2 mean of the finer level (encoder down path)
//   CONV_CAT    [nearest x2 upsample of the coarser level, skip] (decoder)
//   CONV_PLAIN  the map itself (the head; in the bf16 plan also the encoders
//               >= 1, whose input is the 2x2-mean copy the previous encoder's
//               epilogue wrote)
// The epilogue adds the bias and applies ReLU, or for the head the weight
// activation (softplus or exp) on channels 0..M-1 and nothing on the logits.
//
// Three arithmetic forms:
//   fp32: v_mfma_f32_16x16x4f32; LDS holds channel planes so that the 16
//         pixels x 4 channels of an A fragment are bank-conflict free.
//   bf16: v_mfma_f32_16x16x32_bf16; LDS holds pixels with 8-channel runs so
//         that each lane reads its A fragment with one 16-byte load.
//   fp8:  v_mfma_f32_16x16x128_f8f6f4 on e4m3 operands (bf16 activations in
//         memory, quantised with the layer's input scale while staging).
//   All accumulate in fp32.
#include "conv_device.h"

namespace wskp {

template <int EPI>
constexpr bool kHead = EPI == EPI_HEAD_SOFTPLUS || EPI == EPI_HEAD_EXP;

// =============================================================================
// Staging of one reduction chunk: the (TH+KS-1) x (32+KS-1) input halo
// (virtual channels [cc*CK, cc*CK+CK)) and the weight slice.  init() computes each
// item's source offsets once; fetch() only issues global loads into
// registers (and, for pooling, averages them); commit() writes the registers
// to LDS.  The main loop fetches chunk cc+1 while the MFMAs of chunk cc run.
// =============================================================================
template <int PREC, int MODE, int CK, int TH, int NB, typename SrcT, int KS>
struct Stage {
    static constexpr bool BF = PREC == 1;       // bf16 operands
    static constexpr bool F8 = PREC == 2;       // fp8 (e4m3) operands, bf16 activations in HBM
    static constexpr int KR = KS / 2;           // halo width
    static constexpr int TW = kConvTW, HP = TH + KS - 1, WP = TW + KS - 1;
    // input items: a 16-byte run of one pixel's channels (PACK: one pixel)
    static constexpr int G = (MODE == CONV_PACK) ? CK : 16 / (int)sizeof(SrcT);
    static constexpr int NG = CK / G;
    static constexpr int TOT = HP * WP * NG;
    static constexpr int IT = (TOT + kThreads - 1) / kThreads;
    static constexpr int RW = (MODE == CONV_PACK) ? (BF || F8 ? 2 : 3) : 1;  // 16-byte words per item
    // LDS geometry
    static constexpr int PL = ((HP * WP - 16 + 31) / 32) * 32 + 16;     // fp32 plane stride
    static constexpr int PS = CK + 8;                                    // bf16 pixel stride (elements)
    static constexpr int PS8 = CK + 16;                                  // fp8 pixel stride (bytes)
    static constexpr int KE = KS * KS * CK;
    static constexpr int NR = KE / 32;                                   // fp8: runs of 32 K values
    static constexpr int NK = F8 ? (NR + 3) / 4 : (BF ? (KE + 31) / 32 : KE / 4);  // MFMAs per chunk
    static constexpr int BS = NB * 16 + ((NB % 2 == 0) ? 16 : 0);        // fp32 weight row stride
    static constexpr int BSK = NK * 32 + 8;                              // bf16 weight row stride
    static constexpr int BSK8 = NK * 128 + 16;                           // fp8 weight row stride (bytes)
    static constexpr int A_BYTES = F8 ? HP * WP * PS8 : (BF ? HP * WP * PS * 2 : CK * PL * 4);
    static constexpr int B_BYTES = F8 ? NB * 16 * BSK8 : (BF ? NB * 16 * BSK * 2 : KE * BS * 4);
    // weight items: 16 bytes of the packed chunk
    static constexpr int WTOT = F8 ? NB * 16 * NK * 8 : (BF ? NB * 16 * (BSK / 8) : KE * NB * 4);
    static constexpr int WIT = (WTOT + kThreads - 1) / kThreads;
    // per-chunk stride of the packed weights, in elements of the packed type, per output channel
    static constexpr int WCHUNK = F8 ? NK * 128 : (BF ? BSK : KE);

    uint4 in[IT][RW];
    uint4 w[WIT];
    int off0[IT], off1[IT];   // element offsets of the item in source 0 / source 1
    unsigned live;            // bit k: item k lies inside the image
    int woff[WIT];            // element offset of weight item k in chunk 0

    __device__ __forceinline__ void init(const ConvLayer &L, int g, int x0, int y0, int Hl, int Wl)
    {
        const int tid = threadIdx.x;
        live = 0;
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int it = tid + k * kThreads;
            const int p = it / NG, cg = it - p * NG;
            const int ly = p / WP, lx = p - ly * WP;
            const int gy = y0 - KR + ly, gx = x0 - KR + lx;
            off0[k] = off1[k] = 0;
            if (it < TOT && gy >= 0 && gy < Hl && gx >= 0 && gx < Wl) {
                live |= 1u << k;
                if constexpr (MODE == CONV_PACK) {
                    off0[k] = gy * Wl + gx;                                    // pixel index
                } else if constexpr (MODE == CONV_PLAIN) {
                    off0[k] = (gy * Wl + gx) * L.C0 + cg * G;
                } else if constexpr (MODE == CONV_CAT) {
                    off0[k] = ((gy >> 1) * (Wl >> 1) + (gx >> 1)) * L.C0 + cg * G;
                    off1[k] = (gy * Wl + gx) * L.C1 + cg * G;
                } else {  // POOL: top-left of the 2x2 window in the finer level
                    off0[k] = ((2 * gy) * (2 * Wl) + 2 * gx) * L.C0 + cg * G;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < WIT; ++k) {
            const int it = tid + k * kThreads;
            woff[k] = 0;
            if (it < WTOT) {
                if constexpr (F8) {
                    const int co = it / (NK * 8), q = it - co * (NK * 8);
                    woff[k] = (g * NB * 16 + co) * (NK * 128) + q * 16;
                } else if constexpr (BF) {
                    // the group's padded rows are one contiguous block
                    woff[k] = g * NB * 16 * BSK + it * 8;
                } else {
                    const int e = it / (NB * 4), q = it - e * (NB * 4);
                    woff[k] = e * L.Cout_pad + g * NB * 16 + q * 4;
                }
            }
        }
    }

    __device__ __forceinline__ void fetch(const ConvLayer &L, const FrameDesc &fd, const SrcT *s0,
                                          const SrcT *s1, int cc, int Wl)
    {
        const int tid = threadIdx.x;
        const int c0 = cc * CK;
        // decoder input: the whole chunk comes from one source (CK divides C0)
        const bool from_up = (MODE != CONV_CAT) || c0 < L.C0;
        // network input: the raw values of every item (items outside the
        // image read pixel 0 and are zeroed below) are loaded first
        float raw[MODE == CONV_PACK ? IT : 1][10];
        if constexpr (MODE == CONV_PACK) {
#pragma unroll
            for (int k = 0; k < IT; ++k) pack_load(fd, (size_t)off0[k], raw[k]);
        }
#pragma unroll
        for (int k = 0; k < IT; ++k) {
#pragma unroll
            for (int q = 0; q < RW; ++q) in[k][q] = make_uint4(0, 0, 0, 0);
            if (!((live >> k) & 1u)) continue;
            if constexpr (MODE == CONV_PACK) {
                float *x = raw[k];
                pack_transform(L, x);
                if constexpr (F8) {
                    unsigned q[3];
#pragma unroll
                    for (int j = 0; j < 3; ++j) q[j] = fp8x4(x[4 * j] * L.in_qscale, x[4 * j + 1] * L.in_qscale,
                                                       j < 2 ? x[4 * j + 2] * L.in_qscale : 0.f,
                                                       j < 2 ? x[4 * j + 3] * L.in_qscale : 0.f);
                    in[k][0] = make_uint4(q[0], q[1], q[2], 0);
                    in[k][1] = make_uint4(0, 0, 0, 0);
                } else if constexpr (BF) {
                    in[k][0] = make_uint4(pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]),
                                          pack2(x[6], x[7]));
                    in[k][1] = make_uint4(pack2(x[8], x[9]), 0, 0, 0);
                } else {
                    in[k][0] = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]),
                                          __float_as_uint(x[2]), __float_as_uint(x[3]));
                    in[k][1] = make_uint4(__float_as_uint(x[4]), __float_as_uint(x[5]),
                                          __float_as_uint(x[6]), __float_as_uint(x[7]));
                    in[k][2] = make_uint4(__float_as_uint(x[8]), __float_as_uint(x[9]), 0, 0);
                }
            } else if constexpr (MODE == CONV_PLAIN) {
                in[k][0] = gload16(s0 + off0[k] + c0);
            } else if constexpr (MODE == CONV_CAT) {
                in[k][0] = from_up ? gload16(s0 + off0[k] + c0) : gload16(s1 + off1[k] + (c0 - L.C0));
            } else {  // CONV_POOL: 2x2 mean of the finer level
                const SrcT *b = s0 + off0[k] + c0;
                const size_t rs = (size_t)(2 * Wl) * L.C0;
                const uint4 q0 = gload16(b);
                const uint4 q1 = gload16(b + L.C0);
                const uint4 q2 = gload16(b + rs);
                const uint4 q3 = gload16(b + rs + L.C0);
                if constexpr (BF || F8) {
                    const unsigned *a0 = &q0.x, *a1 = &q1.x, *a2 = &q2.x, *a3 = &q3.x;
                    unsigned o[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float lo = 0.25f * (bf16_to_f32(a0[j] & 0xffff) + bf16_to_f32(a1[j] & 0xffff) +
                                                  bf16_to_f32(a2[j] & 0xffff) + bf16_to_f32(a3[j] & 0xffff));
                        const float hi = 0.25f * (bf16_to_f32(a0[j] >> 16) + bf16_to_f32(a1[j] >> 16) +
                                                  bf16_to_f32(a2[j] >> 16) + bf16_to_f32(a3[j] >> 16));
                        o[j] = pack2(lo, hi);
                    }
                    in[k][0] = make_uint4(o[0], o[1], o[2], o[3]);
                } else {
                    const float *f0 = reinterpret_cast<const float *>(&q0), *f1 = reinterpret_cast<const float *>(&q1);
                    const float *f2 = reinterpret_cast<const float *>(&q2), *f3 = reinterpret_cast<const float *>(&q3);
                    float o[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[j] = 0.25f * (f0[j] + f1[j] + f2[j] + f3[j]);
                    in[k][0] = make_uint4(__float_as_uint(o[0]), __float_as_uint(o[1]),
                                          __float_as_uint(o[2]), __float_as_uint(o[3]));
                }
            }
        }
        // weight slice of this chunk
        using WT = typename std::conditional<F8, unsigned char,
                   typename std::conditional<BF, unsigned short, float>::type>::type;
        const WT *wsrc = reinterpret_cast<const WT *>(L.w) + (size_t)cc * WCHUNK * L.Cout_pad;
#pragma unroll
        for (int k = 0; k < WIT; ++k)
            if (tid + k * kThreads < WTOT) w[k] = gload16(wsrc + woff[k]);
    }

    __device__ __forceinline__ void commit(void *As_, void *Bs_, float qs) const
    {
        const int tid = threadIdx.x;
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int it = tid + k * kThreads;
            if (it >= TOT) continue;
            const int p = it / NG, cg = it - p * NG;
            if constexpr (F8) {
                unsigned char *As = static_cast<unsigned char *>(As_);
                if constexpr (MODE == CONV_PACK) {
                    *reinterpret_cast<uint4 *>(&As[p * PS8]) = in[k][0];
                    *reinterpret_cast<uint4 *>(&As[p * PS8 + 16]) = in[k][1];
                } else {
                    // 8 bf16 channels -> 8 scaled e4m3 bytes
                    const unsigned *v = &in[k][0].x;
                    uint2 o;
                    o.x = fp8x4(bf16_to_f32(v[0] & 0xffff) * qs, bf16_to_f32(v[0] >> 16) * qs,
                                bf16_to_f32(v[1] & 0xffff) * qs, bf16_to_f32(v[1] >> 16) * qs);
                    o.y = fp8x4(bf16_to_f32(v[2] & 0xffff) * qs, bf16_to_f32(v[2] >> 16) * qs,
                                bf16_to_f32(v[3] & 0xffff) * qs, bf16_to_f32(v[3] >> 16) * qs);
                    *reinterpret_cast<uint2 *>(&As[p * PS8 + cg * 8]) = o;
                }
            } else if constexpr (BF) {
                unsigned short *As = static_cast<unsigned short *>(As_);
#pragma unroll
                for (int q = 0; q < RW; ++q)
                    *reinterpret_cast<uint4 *>(&As[p * PS + cg * G + q * 8]) = in[k][q];
            } else {
                float *As = static_cast<float *>(As_);
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    const unsigned *v = &in[k][q].x;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int ch = cg * G + q * 4 + j;
                        if (ch < CK) As[ch * PL + p] = __uint_as_float(v[j]);
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < WIT; ++k) {
            const int it = tid + k * kThreads;
            if (it >= WTOT) continue;
            if constexpr (F8) {
                const int co = it / (NK * 8), q = it - co * (NK * 8);
                *reinterpret_cast<uint4 *>(static_cast<unsigned char *>(Bs_) + co * BSK8 + q * 16) = w[k];
            } else if constexpr (BF) {
                *reinterpret_cast<uint4 *>(static_cast<unsigned short *>(Bs_) + it * 8) = w[k];
            } else {
                const int e = it / (NB * 4), q = it - e * (NB * 4);
                *reinterpret_cast<uint4 *>(static_cast<float *>(Bs_) + e * BS + q * 4) = w[k];
            }
        }
    }
};

// The head's weight rows enter the MFMA in the order 0, 4, 8, 12, 1, 5, ...: row
// 4 q + k of the product is channel 4 k + q, so that register k of every lane
// holds channels 4 k .. 4 k + 3 and the epilogue evaluates the weight activation
// for ceil(M / 4) registers instead of all four, and skips those past 2M.
template <bool HEAD>
__device__ __forceinline__ int weight_row(int lj)
{
    return HEAD ? ((lj & 3) << 2) | (lj >> 2) : lj;
}

// One chunk's MFMAs.  fp32: KS*KS*CK/4 steps of v_mfma_f32_16x16x4f32 (K
// order tap, channel); bf16: NK steps of v_mfma_f32_16x16x32_bf16, each
// covering 32 consecutive K values as 4 runs of 8 channels (a run never
// crosses a tap because CK is a multiple of 8; for CK = 16 one MFMA spans
// two taps).
template <int PREC, int MODE, bool HEAD, int CK, int TH, int NB, typename SrcT, int KS>
__device__ __forceinline__ void chunk_mfma(const void *As_, const void *Bs_, f32x4 (*acc)[NB])
{
    using S = Stage<PREC, MODE, CK, TH, NB, SrcT, KS>;
    constexpr int MB = TH / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lj = lane & 15, lq = lane >> 4, lw = weight_row<HEAD>(lj);
    if constexpr (PREC == 0) {
        const float *As = static_cast<const float *>(As_);
        const float *Bs = static_cast<const float *>(Bs_);
#pragma unroll
        for (int tap = 0; tap < KS * KS; ++tap) {
            const int dy = tap / KS, dx = tap % KS;
#pragma unroll
            for (int c4 = 0; c4 < CK / 4; ++c4) {
                float b[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) b[nb] = Bs[(tap * CK + c4 * 4 + lq) * S::BS + nb * 16 + lw];
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const int blk = wave * MB + i, row = blk >> 1, cb = blk & 1;
                    const float a = As[(c4 * 4 + lq) * S::PL + (row + dy) * S::WP + cb * 16 + lj + dx];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[nb], a, acc[i][nb], 0, 0, 0);
                }
            }
        }
    } else if constexpr (PREC == 2) {
        // v_mfma_f32_16x16x128_f8f6f4: lane (i, q) holds 32 consecutive K
        // values (one run of 32 channels of one tap); one MFMA = 4 runs.
        const unsigned char *As = static_cast<const unsigned char *>(As_);
        const unsigned char *Bs = static_cast<const unsigned char *>(Bs_);
#pragma unroll
        for (int s = 0; s < S::NK; ++s) {
            const int run = 4 * s + lq;
            const int k0 = run * 32;
            const int tap = k0 / CK, c0 = k0 - tap * CK;
            const bool live = run < S::NR;
            const int dy = live ? tap / KS : 0, dx = live ? tap % KS : 0;
            i32x8 b[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const unsigned char *bp = &Bs[(nb * 16 + lw) * S::BSK8 + s * 128 + lq * 32];
                const uint4 u0 = *reinterpret_cast<const uint4 *>(bp);
                const uint4 u1 = *reinterpret_cast<const uint4 *>(bp + 16);
                b[nb] = i32x8{(int)u0.x, (int)u0.y, (int)u0.z, (int)u0.w,
                              (int)u1.x, (int)u1.y, (int)u1.z, (int)u1.w};
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int blk = wave * MB + i, row = blk >> 1, cb = blk & 1;
                const int p = (row + dy) * S::WP + cb * 16 + lj + dx;
                const unsigned char *ap = &As[p * S::PS8 + (live ? c0 : 0)];
                uint4 u0 = *reinterpret_cast<const uint4 *>(ap);
                uint4 u1 = *reinterpret_cast<const uint4 *>(ap + 16);
                if (!live) u0 = u1 = make_uint4(0, 0, 0, 0);
                const i32x8 a = i32x8{(int)u0.x, (int)u0.y, (int)u0.z, (int)u0.w,
                                      (int)u1.x, (int)u1.y, (int)u1.z, (int)u1.w};
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[i][nb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        b[nb], a, acc[i][nb], 0, 0, 0, 0, 0, 0);
            }
        }
    } else {
        const unsigned short *As = static_cast<const unsigned short *>(As_);
        const unsigned short *Bs = static_cast<const unsigned short *>(Bs_);
#pragma unroll
        for (int s = 0; s < S::NK; ++s) {
            const int k0 = s * 32 + lq * 8;
            const int tap = k0 / CK, c0 = k0 - tap * CK;
            const bool live = tap < KS * KS;
            const int dy = live ? tap / KS : 0, dx = live ? tap % KS : 0;
            bf16x8 b[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                b[nb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&Bs[(nb * 16 + lw) * S::BSK + k0]));
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int blk = wave * MB + i, row = blk >> 1, cb = blk & 1;
                const int p = (row + dy) * S::WP + cb * 16 + lj + dx;
                u16x8 q = *reinterpret_cast<const u16x8 *>(&As[p * S::PS + (live ? c0 : 0)]);
                if (!live) q = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
                const bf16x8 a = __builtin_bit_cast(bf16x8, q);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[nb], a, acc[i][nb], 0, 0, 0);
            }
        }
    }
}

// Epilogue shared by the conv kernels.  The MFMAs take the weights as their
// first operand, so in output block (i, nb) lane (j, q) holds pixel j of the
// block and the 4 consecutive output channels nb*16 + 4q .. 4q+3.  Bias (and
// the fp8 dequantisation factor) and the activation are applied in
// registers.  Activations (bf16 or fp32 NHWC): each lane writes its 4
// channels with one 8- or 16-byte store; the 4 lanes of a pixel cover 16
// contiguous channels.  The head record (fp32) is planar [2M][H][W], the
// layout the decode reads one map at a time.
//
// With L.pool_idx >= 0 (bf16 activations, a wave owning whole row pairs:
// TH >= 8) the epilogue also writes the 2x2 means of the stored (rounded)
// values to the next level, summed in the order (2y,2x), (2y,2x+1),
// (2y+1,2x), (2y+1,2x+1): the column partner is the neighbouring lane, the
// row partner is block i+2 of the same lane.
// Per-lane output-channel constants of the epilogue: the bias and, for fp8,
// the dequantisation factor of this lane's 4 channels in each block.
template <int PREC, int NB, bool HEAD>
struct EpiConsts {
    float bias[NB][4], dq[NB][4];
    __device__ __forceinline__ void load(const ConvLayer &L, int g)
    {
        const int lq = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int co = g * NB * 16 + nb * 16 + (HEAD ? 4 * v + lq : 4 * lq + v);
                bias[nb][v] = co < L.Cout ? gload(L.bias + co) : 0.f;
                dq[nb][v] = (PREC == 2 && co < L.Cout) ? gload(L.out_scale + co) : 1.f;
            }
    }
};

template <int PREC, int EPI, int TH, int NB, typename OutT>
__device__ __forceinline__ void conv_epilogue(const ConvLayer &L, const FrameDesc &fd, int g, int x0,
                                              int y0, int Hl, int Wl, f32x4 (*acc)[NB],
                                              const EpiConsts<PREC, NB, kHead<EPI>> &ec)
{
    constexpr int MB = TH / 2;
    constexpr int NC = NB * 16;
    constexpr bool CAN_POOL = !std::is_same<OutT, float>::value && EPI == EPI_RELU && MB >= 4 && PREC == 1;
    // bf16 activations of an even number of blocks: stored in pairs
    constexpr bool PAIR = !std::is_same<OutT, float>::value && EPI == EPI_RELU && NB % 2 == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lj = lane & 15, lq = lane >> 4;
    OutT *dst = conv_dst<OutT>(L, fd);
    const bool pool = CAN_POOL && L.pool_idx >= 0;
    OutT *pdst = pool ? reinterpret_cast<OutT *>(fd.p[L.pool_idx]) : nullptr;
    const auto &bias = ec.bias;
    const auto &dq = ec.dq;
    float pe[CAN_POOL ? 2 : 1][CAN_POOL ? NB : 1][4];   // even-row partial sums
    const size_t P = (size_t)Hl * Wl;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int blk = wave * MB + i, row = blk >> 1, cb = blk & 1;
        const int y = y0 + row, x = x0 + cb * 16 + lj;
        const bool in = y < Hl && x < Wl;
        OutT *pp = dst + ((size_t)y * Wl + x) * L.Cout;
        uint2 qs[NB];   // packed bf16 of each block (paired stores)
        uint2 pm[NB];   // packed 2x2 means of each block (odd rows, paired stores)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if constexpr (kHead<EPI>) {
                // head record (one block), planar [2M][H][W]: the 16 lanes of
                // a channel write 16 consecutive pixels of its plane
                OutT *q = dst + lq * P + (unsigned)(y * Wl + x);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (4 * k >= L.Cout) break;
                    float v = acc[i][nb][k] * dq[nb][k] + bias[nb][k];
                    if (4 * k < L.M) v = epilogue<EPI>(v, 4 * k + lq, L.M);
                    if (in && 4 * k + lq < L.Cout) gstore(q + 4 * k * P, v);
                }
                continue;
            }
            const int co = g * NC + nb * 16 + 4 * lq;
            const bool cin = co < L.Cout;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = epilogue<EPI>(acc[i][nb][k] * dq[nb][k] + bias[nb][k], co + k, L.M);
            if constexpr (std::is_same<OutT, float>::value) {
                // fp32 activations: Cout is a multiple of 16
                if (in && cin) gstore(reinterpret_cast<gf32x4 *>(pp + co), gf32x4{v[0], v[1], v[2], v[3]});
            } else {
                // activations: Cout is a multiple of 16
                const uint2 q = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
                qs[nb] = q;
                if constexpr (!PAIR) {
                    if (in && cin) gstore(reinterpret_cast<gu32x2 *>(pp + co), gu32x2{q.x, q.y});
                }
                if constexpr (CAN_POOL) {
                    if (pool) {
                        const float r[4] = {__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xffff0000u),
                                            __uint_as_float(q.y << 16), __uint_as_float(q.y & 0xffff0000u)};
                        const bool odd_row = (i >> 1) & 1;
                        if (!odd_row) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) pe[cb][nb][k] = r[k] + lane_xor1(r[k]);
                        } else {
                            float m[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) m[k] = 0.25f * ((pe[cb][nb][k] + r[k]) + lane_xor1(r[k]));
                            pm[nb] = make_uint2(pack2(m[0], m[1]), pack2(m[2], m[3]));
                            if constexpr (!PAIR) {
                                const int Y = y >> 1, X = x >> 1;
                                if ((lj & 1) == 0 && Y < (Hl >> 1) && X < (Wl >> 1) && cin) {
                                    OutT *pd = pdst + ((size_t)Y * (Wl >> 1) + X) * L.Cout + co;
                                    gstore(reinterpret_cast<gu32x2 *>(pd), gu32x2{pm[nb].x, pm[nb].y});
                                }
                            }
                        }
                    }
                }
            }
        }
        if constexpr (PAIR) {
            // Blocks nb and nb+1 together: lane row q holds channels 4q..4q+3
            // of each.  v_permlane16_swap exchanges the odd rows of the first
            // operand with the even rows of the second, after which even rows
            // hold 8 consecutive channels of block nb (from rows q, q+1) and
            // odd rows 8 of block nb+1 (rows q-1, q): one 16-byte store per
            // lane, and the 4 lanes of a pixel cover its 32 channels.
#pragma unroll
            for (int nb = 0; nb < NB; nb += 2) {
                const auto s0 = __builtin_amdgcn_permlane16_swap(qs[nb].x, qs[nb + 1].x, false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap(qs[nb].y, qs[nb + 1].y, false, false);
                const int c = g * NC + ((lq & 1) ? (nb + 1) * 16 + 4 * (lq - 1) : nb * 16 + 4 * lq);
                if (in && c < L.Cout)
                    gstore(reinterpret_cast<gu32x4 *>(pp + c), gu32x4{s0[0], s1[0], s0[1], s1[1]});
                if constexpr (CAN_POOL) {
                    // the 2x2 means of a row pair, the same way (even lanes)
                    if (pool && ((i >> 1) & 1)) {
                        const auto t0 = __builtin_amdgcn_permlane16_swap(pm[nb].x, pm[nb + 1].x, false, false);
                        const auto t1 = __builtin_amdgcn_permlane16_swap(pm[nb].y, pm[nb + 1].y, false, false);
                        const int Y = y >> 1, X = x >> 1;
                        if ((lj & 1) == 0 && Y < (Hl >> 1) && X < (Wl >> 1) && c < L.Cout) {
                            OutT *pd = pdst + ((size_t)Y * (Wl >> 1) + X) * L.Cout + c;
                            gstore(reinterpret_cast<gu32x4 *>(pd), gu32x4{t0[0], t1[0], t0[1], t1[1]});
                        }
                    }
                }
            }
        }
    }
}

template <int PREC, int MODE, int EPI, int TH, int CK, int NB, typename SrcT, typename OutT, int KS = 3>
__global__ __launch_bounds__(kThreads, (MODE == CONV_PACK && PREC == 1 && KS == 3) ? 4 : 1) void conv3x3_kernel(ConvLayer L, FrameArg fa)
{
    using S = Stage<PREC, MODE, CK, TH, NB, SrcT, KS>;
    constexpr int MB = TH / 2;
    constexpr int LDS_BYTES = S::A_BYTES + S::B_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
    void *As = smem;
    void *Bs = smem + S::A_BYTES;

    int f, g, x0, y0, Hl, Wl;
    if (!conv_locate<TH>(L, fa, f, g, x0, y0, Hl, Wl)) return;
    const FrameDesc &fd = frame_at(fa, f);
    const SrcT *s0 = reinterpret_cast<const SrcT *>(conv_src0(L, fd));
    const SrcT *s1 = reinterpret_cast<const SrcT *>(fd.e[L.src1_idx]);
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    S st;
    st.init(L, g, x0, y0, Hl, Wl);
    const int nchunks = L.Cin_pad / CK;
    st.fetch(L, fd, s0, s1, 0, Wl);
    EpiConsts<PREC, NB, kHead<EPI>> ec;
    if constexpr (MODE == CONV_PACK) {
        // the network input is one chunk: the epilogue's constants are
        // requested once the staged values are in LDS (their registers are
        // free again) and the MFMAs hide their latency; the barrier waits for
        // LDS only, not for these loads
        st.commit(As, Bs, L.in_qscale);
        ec.load(L, g);
        lds_sync();
        chunk_mfma<PREC, MODE, kHead<EPI>, CK, TH, NB, SrcT, KS>(As, Bs, acc);
    } else {
        for (int cc = 0; cc < nchunks; ++cc) {
            if (cc) __syncthreads();
            st.commit(As, Bs, L.in_qscale);
            __syncthreads();
            if (cc + 1 < nchunks) st.fetch(L, fd, s0, s1, cc + 1, Wl);
            chunk_mfma<PREC, MODE, kHead<EPI>, CK, TH, NB, SrcT, KS>(As, Bs, acc);
        }
        ec.load(L, g);
    }

    conv_epilogue<PREC, EPI, TH, NB, OutT>(L, fd, g, x0, y0, Hl, Wl, acc, ec);
}

// =============================================================================
// bf16 convs of an odd number of output blocks (48, 80 channels, the head) with
// direct-to-LDS buffer loads, one 16-channel block per workgroup; layers of pairs
// of blocks run conv_bf16.hip
// =============================================================================
// Every 16-byte slot of the input halo (8 bf16 channels of one pixel) and of
// the weight slice goes from memory straight into LDS with
// buffer_load_dwordx4 ... lds: no registers hold staged data and no commit
// pass rewrites it.  A wave-level load writes 64 consecutive slots, so the
// LDS image of the halo is pixel-major with 4 slots per pixel (CK = 32
// channels).  A 16-byte LDS read serves 8 lanes per cycle from 32 banks, so
// the 8 pixels a fragment read takes in one cycle must land in 8 distinct
// 16-byte bank groups of a 128-byte line: the 4 slots of pixel p hold channel
// groups in the order g ^ ((p >> 1) & 3), which with the pixel's position
// in the line (p & 1) enumerates all 8 groups for any 8 consecutive pixels.
// Each lane realises the order by choosing which group it fetches.  Pixels outside the image
// get an offset beyond the buffer's range, and the hardware returns zeros:
// that is the conv's zero padding.

#ifndef WSKP_DIRECT_SWZ
#define WSKP_DIRECT_SWZ 1
#endif
constexpr int kDirectSwz = WSKP_DIRECT_SWZ;

__device__ __forceinline__ void load_lds16(rsrc_t r, unsigned char *lds, unsigned voff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16,
                                             (int)voff, 0, 0, 0);
}

constexpr unsigned kOutOfRange = 0x7ffffff0u;

// Each wave computes HW = TH/4 output rows of the tile (both 16-pixel column
// blocks).  For one column offset dx it reads the A
// fragments of its HW+KS-1 input rows once and uses each for up to KS
// vertical taps dy (input row r+dy feeds output row r), so a 3x3 chunk costs
// 6 (HW+2) A fragment reads instead of 18 HW: the LDS bytes per MFMA, which
// bound this loop, fall with HW.
// Workgroups per CU that the stage's LDS (160 KiB per CU) admits, at most
// four (at TH = 8: 3x3, 31 KiB, four; 5x5, 52 KiB, three); the register budget
// is capped to match.
constexpr int direct_stage_bytes(int KS, int TH)
{
    return ((TH + KS - 1) * (kConvTW + KS - 1) * 64 + 16 * KS * KS * 64 + 1023) / 1024 * 1024;
}
constexpr int direct_min_wg(int KS, int TH)
{
    return 163840 / direct_stage_bytes(KS, TH) < 4 ? 163840 / direct_stage_bytes(KS, TH) : 4;
}

template <int MODE, int EPI, int TH, typename OutT, int KS = 3>
__global__ __launch_bounds__(kThreads, direct_min_wg(KS, TH)) void conv3x3_bf16_direct(ConvLayer L, FrameArg fa)
{
    constexpr int CK = 32, WP = kConvTW + KS - 1, HP = TH + KS - 1, NPIX = HP * WP;
    constexpr int A_SLOTS = NPIX * 4;
    constexpr int NK = KS * KS;                            // one tap (32 channels) per MFMA
    // Weight rows are unpadded (k^2 taps x 32 channels: 576 B for 3x3,
    // 1600 B for 5x5); in row co
    // the 16-byte column groups are stored XOR-ed with 2 * ((co >> 2) & 1)
    // (host packing), so the 16 rows x 4 groups of a B-fragment read fall
    // on distinct banks (a 592-byte padded row costs 4 extra LDS cycles per
    // read on gfx950).
    constexpr int BSK = NK * 32;
    constexpr int B_SLOTS = 16 * BSK / 8;
    // The stage is one array of 16-byte slots, halo first, weights right
    // after it; load instruction j fills slots [64j, 64j + 64).  The
    // instruction that straddles the boundary is issued twice, once per
    // source, each with only its own lanes active.
    constexpr int SLOTS = A_SLOTS + B_SLOTS;
    constexpr int INS = (SLOTS + 63) / 64;
    constexpr int PW = (INS + 3) / 4;                      // load instructions per wave
    constexpr int A_BYTES = A_SLOTS * 16, STAGE = INS * 1024;
    static_assert(STAGE == direct_stage_bytes(KS, TH), "stage size");
    constexpr int MB = TH / 2, HW = TH / 4;
    static_assert(TH % 4 == 0, "each wave owns TH/4 whole rows");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGE];

    int f, g, x0, y0, Hl, Wl;
    if (!conv_locate<TH>(L, fa, f, g, x0, y0, Hl, Wl)) return;
    const FrameDesc &fd = frame_at(fa, f);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 15, lq = lane >> 4;
    const int lw = weight_row<kHead<EPI>>(lj);
    const int bq = lq ^ (((lw >> 2) & 1) << 1);   // swizzled weight column group

    const unsigned short *s0 =
        reinterpret_cast<const unsigned short *>(conv_src0(L, fd));
    const unsigned short *s1 = reinterpret_cast<const unsigned short *>(fd.e[L.src1_idx]);
    const int H0 = MODE == CONV_CAT ? Hl >> 1 : Hl, W0 = MODE == CONV_CAT ? Wl >> 1 : Wl;
    const rsrc_t r0 = make_rsrc(s0, (unsigned)((size_t)H0 * W0 * L.C0 * 2));
    const rsrc_t r1 = make_rsrc(s1, MODE == CONV_CAT ? (unsigned)((size_t)Hl * Wl * L.C1 * 2) : 0u);
    const int nchunks = L.Cin_pad / CK;
    const rsrc_t rw = make_rsrc(L.w, (unsigned)((size_t)nchunks * L.Cout_pad * BSK * 2));

    // byte offsets of this wave's A slots in source 0 and source 1 (chunk 0).
    // The lane's k-th slot is slot0 + 256 k: halo pixel p0 + 64 k with the
    // same channel group (adding 64 leaves bits 1-2 of the pixel index
    // unchanged), so its row and column step by the quotient and remainder
    // of 64 / WP.  Row and pixel pitches are below 2^24, so the products are
    // 24-bit multiplies (full rate, unlike 32-bit ones).
    const unsigned cp0 = (unsigned)L.C0 * 2u, rp0 = (unsigned)W0 * cp0;
    const unsigned cp1 = (unsigned)L.C1 * 2u, rp1 = (unsigned)Wl * cp1;
    const int slot0 = wave * 64 + lane, p0 = slot0 >> 2;
    const unsigned goff = (unsigned)(((slot0 & 3) ^ ((p0 >> kDirectSwz) & 3)) * 16);
    constexpr int SY = 64 / WP, SX = 64 - SY * WP;
    int ly = p0 / WP, lx = p0 - ly * WP;
    unsigned oa0[PW], oa1[PW];
#pragma unroll
    for (int k = 0; k < PW; ++k) {
        const int gy = y0 - KS / 2 + ly, gx = x0 - KS / 2 + lx;
        const bool in = p0 + 64 * k < NPIX && (unsigned)gy < (unsigned)Hl && (unsigned)gx < (unsigned)Wl;
        if (MODE == CONV_CAT) {
            oa0[k] = in ? __umul24((unsigned)gy >> 1, rp0) + __umul24((unsigned)gx >> 1, cp0) + goff : kOutOfRange;
            oa1[k] = in ? __umul24((unsigned)gy, rp1) + __umul24((unsigned)gx, cp1) + goff : kOutOfRange;
        } else {
            oa0[k] = in ? __umul24((unsigned)gy, rp0) + __umul24((unsigned)gx, cp0) + goff : kOutOfRange;
            oa1[k] = kOutOfRange;
        }
        lx += SX;
        ly += SY;
        if (lx >= WP) {
            lx -= WP;
            ++ly;
        }
    }

    // issues chunk cc's halo and weight slices into the stage at `buf`
    auto issue = [&](int cc, unsigned char *buf) {
        const int c0 = cc * CK;
        const bool up = MODE != CONV_CAT || c0 < L.C0;
        const unsigned da = (unsigned)((up ? c0 : c0 - L.C0) * 2);
        const unsigned wb = (unsigned)((cc * L.Cout_pad + g * 16) * BSK * 2);
#pragma unroll
        for (int k = 0; k < PW; ++k) {
            const int ins = wave + 4 * k;
            if (ins >= INS) break;
            const int slot = ins * 64 + lane;
            unsigned char *dst = buf + ins * 1024;
            if (ins * 64 < A_SLOTS && slot < A_SLOTS) {
                if (up) load_lds16(r0, dst, oa0[k] + da);
                else load_lds16(r1, dst, oa1[k] + da);
            }
            if (ins * 64 + 64 > A_SLOTS && slot >= A_SLOTS && slot < SLOTS)
                load_lds16(rw, dst, wb + (unsigned)((slot - A_SLOTS) * 16));
        }
    };

    f32x4 acc[MB][1];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i][0] = f32x4{0.f, 0.f, 0.f, 0.f};

    // MFMAs of one chunk from the stage at As (halo) / As + A_BYTES (weights)
    auto compute = [&](const unsigned char *As) {
        const unsigned char *Bs = As + A_BYTES;
#pragma unroll
        for (int dx = 0; dx < KS; ++dx) {
            bf16x8 a[HW + KS - 1][2];
#pragma unroll
            for (int rr = 0; rr < HW + KS - 1; ++rr)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const int p = (wave * HW + rr) * WP + cb * 16 + lj + dx;
                    const int slot = p * 4 + (lq ^ ((p >> kDirectSwz) & 3));
                    a[rr][cb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(As + slot * 16));
                }
#pragma unroll
            for (int dy = 0; dy < KS; ++dy) {
                const int s = dy * KS + dx;
                const bf16x8 b = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u16x8 *>(Bs + (lw * BSK + s * 32 + bq * 8) * 2));
#pragma unroll
                for (int r = 0; r < HW; ++r)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
                        acc[2 * r + cb][0] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[r + dy][cb], acc[2 * r + cb][0], 0, 0, 0);
            }
        }
    };

    issue(0, smem);
    for (int cc = 0; cc < nchunks; ++cc) {
        wait_vmem<0>();
        lds_barrier();
        compute(smem);
        wait_lds();
        lds_barrier();   // the stage has been read before it is refilled
        if (cc + 1 < nchunks) issue(cc + 1, smem);
    }
    EpiConsts<1, 1, kHead<EPI>> ec;
    ec.load(L, g);
    conv_epilogue<1, EPI, TH, 1, OutT>(L, fd, g, x0, y0, Hl, Wl, acc, ec);
}

// =============================================================================
// dispatch
// =============================================================================
// Output rows per conv tile (build-time tuning knobs): kTH for the kernels
// that stage through registers, kTHD (a multiple of 4) for the direct-load
// bf16 kernel.
#ifndef WSKP_CONV_TH
#define WSKP_CONV_TH 4
#endif
#ifndef WSKP_DIRECT_TH
#define WSKP_DIRECT_TH 8
#endif
#ifndef WSKP_CONV_DIRECT
#define WSKP_CONV_DIRECT 1
#endif
constexpr int kTH = WSKP_CONV_TH;
// fp8: 8 rows, so that a weight fragment read from LDS serves four blocks of 16
// pixels instead of two and the halo is a third instead of half of the tile; its time
// goes to LDS reads and the quantisation while staging.  1080p, four levels:
// 632 us with 4 rows, 557 with 8 (the full-resolution decoder 150 -> 127, the head
// 94 -> 76, the widest decoder 105 -> 82).
constexpr int kTH8 = 8;
// the network-input layer (one reduction chunk) gets its own knob
#ifndef WSKP_PACK_TH
#define WSKP_PACK_TH 8
#endif
constexpr int kTHP = WSKP_PACK_TH;
constexpr int kTHD = WSKP_DIRECT_TH;

static bool uses_direct(int prec, int mode, int CK, int ks)
{
    return WSKP_CONV_DIRECT && (ks == 3 || ks == 5) && prec == 1 && CK == 32 &&
           (mode == CONV_CAT || mode == CONV_PLAIN);
}

bool conv_uses_direct(int prec, int mode, int CK, int ks) { return uses_direct(prec, mode, CK, ks); }

// Tile rows per layer: the input layer uses kTHP; the direct-load kernel uses
// kTHD, or 4 rows on the levels from WSKP_COARSE_LEVEL on, which have few
// pixels, so that they still spread over all CUs, unless the layer passes on
// 2x2 means (that needs whole row pairs per wave, 8 rows).  From level 4: with
// level 3 on 4-row tiles too (the fourth level of the 720p net, 160 x 90) one
// frame's launch was slightly faster alone but three-stream throughput 1 %
// lower.  (Layers of conv_bf16.hip choose theirs for each launch, and so do
// fp32 and fp8 layers.)
#ifndef WSKP_COARSE_LEVEL
#define WSKP_COARSE_LEVEL 4
#endif
int conv_tile_rows(int prec, int mode, int CK, int level, bool pool, int ks)
{
    if (mode == CONV_PACK) return kTHP;
    if (!uses_direct(prec, mode, CK, ks)) return prec == 2 ? kTH8 : kTH;
    return (level >= WSKP_COARSE_LEVEL && !pool) ? 4 : kTHD;
}

int conv_chunk(int prec, int mode, int Cin, int C0)
{
    if (prec == 2) return 32;   // fp8: runs of 32 channels (the network input padded to 32)
    if (mode == CONV_PACK) return prec == 0 ? 12 : 16;
    if (prec != 0 && Cin % 32 == 0 && (mode != CONV_CAT || C0 % 32 == 0)) return 32;
    return 16;
}

#ifndef WSKP_CONV_MAX_NB
#define WSKP_CONV_MAX_NB 4
#endif
// Wider groups stage and read each input tile fewer times (the A operand is
// reused across NB blocks); narrower groups give more workgroups and a
// smaller stage, so more of them fit a CU.  5x5 layers of the register-staged
// kernel take one block per group: their weight slices are 25/9 times larger.
int conv_blocks_per_group(int prec, int mode, int CK, int nblk, int ks)
{
    // pairs of blocks run conv_bf16.hip
    if (uses_direct(prec, mode, CK, ks)) return nblk % 2 == 0 ? 2 : 1;
    if (ks != 3) return 1;
    if (mode == CONV_PACK) return nblk % 2 == 0 ? 2 : 1;
    for (int nb = WSKP_CONV_MAX_NB; nb > 1; --nb)
        if (nb <= 4 && nblk % nb == 0) return nb;
    return 1;
}

int conv_grid(const ConvLayer &L, int n, const int *H, const int *W)
{
    long total = 0;
    for (int f = 0; f < n; ++f) {
        const int Hl = H[f] >> L.level, Wl = W[f] >> L.level;
        total += (long)((Wl + kConvTW - 1) / kConvTW) * ((Hl + L.th - 1) / L.th) * L.groups;
    }
    return (int)total;
}

// FP32 layers of few pixels: a workgroup's time is its serial chain of MFMAs
// (32 cycles each, TH/2 NB of them per four input channels and tap), so
// below two workgroups per CU first the output blocks of a workgroup, then its
// rows are cut: at (2 rows, 1 block) the chain is an eighth of that at (4, 4).
// A wider grid costs re-reads of the input tile and of the halo, which pay only
// while CUs are idle.  The weights' layout and every output's order of
// summation do not depend on the tiling.  The small net, us at 16x16 / 128x128 /
// 256x256 / 320x400: 69 / 74 / 81 / 125 without the rule, 41 / 43 / 61 / 109 at
// this line, 41 / 43 / 62 / 120 at 256 workgroups, 41 / 43 / 61 / 110 at 1024; the
// 4-level net at 64x64 / 256x256: 235 / 270 -> 90 / 176.  A training step of
// 8 crops of 256x256 is 1 % slower at 1024 than here, 3 % at 2048.
constexpr int kFp32Grid = 512;

// Decoders of two or four blocks per group take 8-row tiles where enough of them
// are left: each weight fragment read from LDS serves four blocks of 16 pixels
// instead of two.  8 crops of 256x256: 96 -> 32 channels 264 -> 240 us, 160 -> 64
// 198 -> 188.  The encoders, one block and three blocks measured slower so (registers:
// one wave fewer per SIMD).
static bool fp32_tall(const ConvLayer &L) { return L.ks == 3 && L.C1 > 0 && (L.NB == 2 || L.NB == 4); }

int conv_fp32_tiles(ConvLayer &L, int n, const int *H, const int *W)
{
    int blocks = conv_grid(L, n, H, W);
    const int nblk = L.Cout_pad / 16;
    if (fp32_tall(L)) {
        ConvLayer t = L;
        t.th = 8;
        const int b = conv_grid(t, n, H, W);
        if (b >= kFp32Grid) {
            L.th = 8;
            return b;
        }
    }
    while (blocks < kFp32Grid && L.NB > 1) {
        do --L.NB;
        while (nblk % L.NB);
        L.groups = nblk / L.NB;
        blocks = conv_grid(L, n, H, W);
    }
    while (blocks < kFp32Grid && L.th > 2) {
        L.th /= 2;
        blocks = conv_grid(L, n, H, W);
    }
    return blocks;
}

// fp8: 4-row tiles where 8-row ones leave most CUs with a single workgroup and its
// serial chain of chunks: up to one for each CU, or up to 1.5 where a workgroup has
// one or two output blocks (4 rows / 8 rows, us: the 4-level net at 208x384, 312
// tiles at full resolution, 98 / 100; 64 and 128 channels at 272x480, 272 tiles of
// four blocks at half resolution, 79 / 76).  The 4-level net with 8 rows / 4 rows / this
// rule: 64x96 99 / 80 / 80, 256x256 111 / 92 / 90, 360x640 141 / 126 / 127,
// 720x1280 275 / 310 / 272, 1080x1920 554 / 633 / 554.  Every output's order of
// summation is the same.
int conv_fp8_rows(const ConvLayer &L, int mode, int n, const int *H, const int *W)
{
    return mode != CONV_PACK && conv_grid(L, n, H, W) <= (L.NB > 2 ? 256 : 384) ? 4 : L.th;
}

// The cut tiles of conv_fp32_tiles: TH rows, one block.
template <int MODE, int EPI, int TH, int CK>
static bool launch_fp32_small(const ConvLayer &L, const FrameArg &fa, int blocks, hipStream_t s)
{
    if (L.th != TH) return false;
    if (L.ks == 5)
        hipLaunchKernelGGL((conv3x3_kernel<0, MODE, EPI, TH, CK, 1, float, float, 5>), dim3(blocks), dim3(kThreads), 0,
                           s, L, fa);
    else
        hipLaunchKernelGGL((conv3x3_kernel<0, MODE, EPI, TH, CK, 1, float, float>), dim3(blocks), dim3(kThreads), 0, s,
                           L, fa);
    return true;
}

template <int PREC, int MODE, int EPI, int CK, int NB, typename OutT>
static void launch_one(const ConvLayer &L, const FrameArg &fa, int blocks, hipStream_t s)
{
    using SrcT = typename std::conditional<PREC == 0, float, unsigned short>::type;
    constexpr int TH = MODE == CONV_PACK ? kTHP : PREC == 2 ? kTH8 : kTH;
    if constexpr (PREC == 0 && MODE == CONV_CAT && (NB == 2 || NB == 4)) {
        if (L.th == 8) {
            hipLaunchKernelGGL((conv3x3_kernel<0, MODE, EPI, 8, CK, NB, float, float>), dim3(blocks), dim3(kThreads), 0,
                               s, L, fa);
            return;
        }
    }
    if constexpr (PREC == 0 && NB == 1) {
        if (launch_fp32_small<MODE, EPI, 2, CK>(L, fa, blocks, s)) return;
        if constexpr (TH == 8)
            if (launch_fp32_small<MODE, EPI, 4, CK>(L, fa, blocks, s)) return;
    }
    if constexpr (WSKP_CONV_DIRECT && NB == 1 && PREC == 1 && CK == 32 && (MODE == CONV_CAT || MODE == CONV_PLAIN)) {
        if (L.ks == 5) {
            if (L.th == 4)
                hipLaunchKernelGGL((conv3x3_bf16_direct<MODE, EPI, 4, OutT, 5>), dim3(blocks), dim3(kThreads), 0, s,
                                   L, fa);
            else
                hipLaunchKernelGGL((conv3x3_bf16_direct<MODE, EPI, kTHD, OutT, 5>), dim3(blocks), dim3(kThreads),
                                   0, s, L, fa);
            return;
        }
    }
    if constexpr (NB == 1 && PREC != 2) {
        if (L.ks == 5) {
            hipLaunchKernelGGL((conv3x3_kernel<PREC, MODE, EPI, TH, CK, NB, SrcT, OutT, 5>), dim3(blocks),
                               dim3(kThreads), 0, s, L, fa);
            return;
        }
    }
    if constexpr (WSKP_CONV_DIRECT && NB == 1 && PREC == 1 && CK == 32 && (MODE == CONV_CAT || MODE == CONV_PLAIN)) {
        if (L.th == 4)
            hipLaunchKernelGGL((conv3x3_bf16_direct<MODE, EPI, 4, OutT>), dim3(blocks),
                               dim3(kThreads), 0, s, L, fa);
        else
            hipLaunchKernelGGL((conv3x3_bf16_direct<MODE, EPI, kTHD, OutT>), dim3(blocks),
                               dim3(kThreads), 0, s, L, fa);
        return;
    }
    if constexpr (PREC == 2 && MODE != CONV_PACK) {
        if (L.th == 4) {
            hipLaunchKernelGGL((conv3x3_kernel<2, MODE, EPI, 4, CK, NB, SrcT, OutT>), dim3(blocks), dim3(kThreads), 0, s,
                               L, fa);
            return;
        }
    }
    // fp32 activations travel with the fp32 MFMA form; the bf16 and fp8 forms
    // keep bf16 activations in memory
    hipLaunchKernelGGL((conv3x3_kernel<PREC, MODE, EPI, TH, CK, NB, SrcT, OutT>), dim3(blocks),
                       dim3(kThreads), 0, s, L, fa);
}

// Chunk sizes: fp32 uses CK = 12 (network input) or 16; bf16 uses 16 (input
// padded from 10) or 32 where the channel counts allow it.
template <int PREC, int MODE, int EPI, typename OutT>
static bool launch_ck_nb(const ConvLayer &L, const FrameArg &fa, int blocks, hipStream_t s)
{
#define WSKP_CASE(ck, nb)                                                   \
    if (L.CK == ck && L.NB == nb) {                                         \
        launch_one<PREC, MODE, EPI, ck, nb, OutT>(L, fa, blocks, s);       \
        return true;                                                        \
    }
    if constexpr (PREC == 2) {
        WSKP_CASE(32, 1) WSKP_CASE(32, 2)
        if constexpr (MODE != CONV_PACK && MODE != CONV_PLAIN) { WSKP_CASE(32, 3) WSKP_CASE(32, 4) }
    } else if constexpr (MODE == CONV_PACK) {
        if constexpr (PREC == 0) { WSKP_CASE(12, 1) WSKP_CASE(12, 2) }
        else { WSKP_CASE(16, 1) WSKP_CASE(16, 2) }
    } else if constexpr (MODE == CONV_PLAIN) {
        WSKP_CASE(16, 1)
        if constexpr (PREC != 0) { WSKP_CASE(32, 1) }
    } else {
        WSKP_CASE(16, 1) WSKP_CASE(16, 2) WSKP_CASE(16, 3) WSKP_CASE(16, 4)
        if constexpr (PREC != 0) { WSKP_CASE(32, 1) }
        if constexpr (PREC == 1 && MODE == CONV_POOL) { WSKP_CASE(32, 2) WSKP_CASE(32, 3) WSKP_CASE(32, 4) }
    }
#undef WSKP_CASE
    return false;
}

template <int PREC>
static bool dispatch(const ConvLayer &L, int mode, int epi, const FrameArg &fa, int blocks,
                     hipStream_t s)
{
    using ActT = typename std::conditional<PREC == 0, float, unsigned short>::type;
    switch (mode) {
    case CONV_PACK: return launch_ck_nb<PREC, CONV_PACK, EPI_RELU, ActT>(L, fa, blocks, s);
    case CONV_POOL: return launch_ck_nb<PREC, CONV_POOL, EPI_RELU, ActT>(L, fa, blocks, s);
    case CONV_CAT: return launch_ck_nb<PREC, CONV_CAT, EPI_RELU, ActT>(L, fa, blocks, s);
    case CONV_PLAIN:
        // encoders on pooled maps (bf16); the head record is fp32 in every precision
        if (epi == EPI_RELU) return launch_ck_nb<PREC, CONV_PLAIN, EPI_RELU, ActT>(L, fa, blocks, s);
        if (epi == EPI_HEAD_EXP) return launch_ck_nb<PREC, CONV_PLAIN, EPI_HEAD_EXP, float>(L, fa, blocks, s);
        return launch_ck_nb<PREC, CONV_PLAIN, EPI_HEAD_SOFTPLUS, float>(L, fa, blocks, s);
    default: return false;
    }
}

hipError_t launch_conv(const ConvLayer &L, int mode, int epi, int prec, const FrameArg &fa,
                       int blocks, hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    // 5x5 layers run the register-staged kernel with one block per group
    if (L.NB == 2 && epi == EPI_RELU && uses_direct(prec, mode, L.CK, L.ks)) return launch_conv_bf16(L, mode, fa, blocks, s);
    if (L.ks != 3 && (L.ks != 5 || L.NB != 1 || prec == 2)) return hipErrorInvalidValue;
    const bool ok = prec == 0   ? dispatch<0>(L, mode, epi, fa, blocks, s)
                    : prec == 1 ? dispatch<1>(L, mode, epi, fa, blocks, s)
                                : dispatch<2>(L, mode, epi, fa, blocks, s);
    if (!ok) return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace wskp
