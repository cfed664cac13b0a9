// Device helpers shared by the convolution kernels (conv3x3.hip,
// conv_split.hip): element conversions, tile lookup, the weight activation
// and the network input's preprocessing.
#pragma once

#include "wskp_internal.h"

#include <type_traits>

namespace wskp {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// ---- element conversions ---------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(unsigned short h)
{
    return __uint_as_float(((unsigned int)h) << 16);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// fp32 -> bf16 with round-to-nearest-even: one v_cvt_pk_bf16_f32 for a pair
__device__ __forceinline__ unsigned cvt_pk_bf16(float a, float b)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

__device__ __forceinline__ unsigned short f32_to_bf16(float f) { return (unsigned short)cvt_pk_bf16(f, 0.f); }

// Three bf16 parts of two values, packed (the first value in the low half):
// v = p0 + p1 + p2, each part the round-to-nearest bf16 of what the parts before
// it leave.  Exact from 2^-110 up (below, the third and then the second part
// runs out of bf16's range).  Infinities and NaNs stay in their first part
// and make the others NaN (see sum_parts).  Finite values above the largest bf16
// would round to infinity: WIDE gives them that for their first part.
constexpr float kBf16Max = 0x1.fep127f;
template <bool WIDE>
__device__ __forceinline__ void split_bf16(float a, float b, unsigned (&p)[3])
{
    auto first = [](float v) {
        return WIDE && fabsf(v) < INFINITY ? __builtin_amdgcn_fmed3f(v, -kBf16Max, kBf16Max) : v;
    };
    p[0] = cvt_pk_bf16(first(a), first(b));
    a -= __uint_as_float(p[0] << 16);
    b -= __uint_as_float(p[0] & 0xffff0000u);
    p[1] = cvt_pk_bf16(a, b);
    a -= __uint_as_float(p[1] << 16);
    b -= __uint_as_float(p[1] & 0xffff0000u);
    p[2] = cvt_pk_bf16(a, b);
}
// 2 N values; the wide form only where a lane of the wave has a value that needs it
// (a maximum over three costs half an instruction a value, the wide form three)
template <int N>
__device__ __forceinline__ void split_bf16_run(const float *v, unsigned (&p)[N][3])
{
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 2 * N; ++e) m = fmaxf(m, fabsf(v[e]));
    if (__builtin_expect(__any(m > kBf16Max), 0)) {
#pragma unroll
        for (int e = 0; e < N; ++e) split_bf16<true>(v[2 * e], v[2 * e + 1], p[e]);
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) split_bf16<false>(v[2 * e], v[2 * e + 1], p[e]);
    }
}
// The sum of a product of split operands from its main accumulator (the
// products of the first parts) and that of the small terms.  Where an
// operand is infinite the small terms are NaN and the main sum is the fp32 one:
// infinite, or NaN for infinities of both signs or times zero.
__device__ __forceinline__ float sum_parts(float main, float small)
{
    const float v = main + small;
    return v == v ? v : main;
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    __device__ static __forceinline__ void load4(const float *p, float v[4])
    {
        const float4 q = *reinterpret_cast<const float4 *>(p);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
    __device__ static __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct Elem<unsigned short> {
    __device__ static __forceinline__ void load4(const unsigned short *p, float v[4])
    {
        const uint2 q = *reinterpret_cast<const uint2 *>(p);
        v[0] = __uint_as_float(q.x << 16);
        v[1] = __uint_as_float(q.x & 0xffff0000u);
        v[2] = __uint_as_float(q.y << 16);
        v[3] = __uint_as_float(q.y & 0xffff0000u);
    }
    __device__ static __forceinline__ void store(unsigned short *p, float v) { *p = f32_to_bf16(v); }
};

// ---- tile lookup -------------------------------------------------------------
// A tile of a conv layer: TH output rows x kConvTW columns at (y0, x0) of the
// layer's level of frame f, output-channel group g; Hl x Wl the level's size.
template <int TH>
struct ConvTile {
    int f, g, x0, y0, Hl, Wl;
    // From logical tile t of frames first .. first + n - 1; false past the
    // last tile.
    __device__ __forceinline__ bool set(const ConvLayer &L, const FrameArg &fa, int first, int n, int t)
    {
        const int lev = L.level, groups = L.groups;
        auto tiles = [=](int H, int W) {
            return (((W >> lev) + kConvTW - 1) / kConvTW) * (((H >> lev) + TH - 1) / TH) * groups;
        };
        f = batch_frame(fa, first, n, t, tiles);
        if (f < 0) return false;
        const FrameDesc &fd = frame_at(fa, f);
        Hl = fd.H >> lev;
        Wl = fd.W >> lev;
        const int txn = (Wl + kConvTW - 1) / kConvTW;
        g = t % groups;
        t /= groups;
        x0 = (t % txn) * kConvTW;
        y0 = (t / txn) * TH;
        return true;
    }
};

// Maps this workgroup to its tile.  Returns false for workgroups beyond the
// batch's tile count (capacity launches).
template <int TH>
__device__ __forceinline__ bool conv_locate(const ConvLayer &L, const FrameArg &fa, int &f, int &g,
                                            int &x0, int &y0, int &Hl, int &Wl)
{
    int first, n;
    const int t = batch_tile_id(fa, blockIdx.x, gridDim.x, first, n);
    ConvTile<TH> c;
    if (t < 0 || !c.set(L, fa, first, n, t)) return false;
    f = c.f;
    g = c.g;
    x0 = c.x0;
    y0 = c.y0;
    Hl = c.Hl;
    Wl = c.Wl;
    return true;
}

// ---- fast transcendental helpers -------------------------------------------
// v_exp_f32 / v_log_f32 compute 2^x and log2(x) to about 1 ulp for normal
// inputs.  log1p uses the compensated form log(u) * t / (u - 1), u = 1 + t,
// which removes the rounding of 1 + t (Goldberg's method), so the result keeps
// full relative accuracy for small t.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

__device__ __forceinline__ float log1p_small(float t)
{
    const float u = 1.f + t;
    if (u == 1.f) return t;
    // t / (u - 1) is 1 up to the rounding of u: the hardware reciprocal
    // (1 ulp) instead of an IEEE division
    return fast_log2(u) * 0.69314718055994531f * (t * __builtin_amdgcn_rcpf(u - 1.f));
}

// softplus(x) = max(x, 0) + log(1 + e^{-|x|})
__device__ __forceinline__ float softplus_f(float x)
{
    const float t = fast_exp2(-fabsf(x) * 1.4426950408889634f);
    return fmaxf(x, 0.f) + log1p_small(t);
}

template <int EPI>
__device__ __forceinline__ float epilogue(float v, int co, int M)
{
    if (EPI == EPI_RELU) return fmaxf(v, 0.f);
    // exp weights: the raw pre-activation is stored; the decode takes the
    // exponential with a per-tile shift (no overflow for any finite h)
    if (co < M && EPI == EPI_HEAD_SOFTPLUS) return softplus_f(v);
    return v;
}

__device__ __forceinline__ const void *conv_src0(const ConvLayer &L, const FrameDesc &fd)
{
    return L.src0_kind == 0 ? fd.e[L.src0_idx] : (L.src0_kind == 1 ? fd.u[L.src0_idx] : fd.p[L.src0_idx]);
}

template <typename OutT>
__device__ __forceinline__ OutT *conv_dst(const ConvLayer &L, const FrameDesc &fd)
{
    if (L.out_kind == 2) return reinterpret_cast<OutT *>(fd.head);
    return reinterpret_cast<OutT *>(L.out_kind ? fd.u[L.out_idx] : fd.e[L.out_idx]);
}

__device__ __forceinline__ unsigned pack2(float a, float b)
{
    return cvt_pk_bf16(a, b);
}

typedef int i32x8 __attribute__((ext_vector_type(8)));

// Four floats -> four OCP e4m3 bytes (round to nearest even), saturated to
// the largest finite magnitude 448 first so that no value becomes NaN.
__device__ __forceinline__ unsigned fp8x4(float a, float b, float c, float d)
{
    const float m = 448.f;
    a = __builtin_amdgcn_fmed3f(a, -m, m);
    b = __builtin_amdgcn_fmed3f(b, -m, m);
    c = __builtin_amdgcn_fmed3f(c, -m, m);
    d = __builtin_amdgcn_fmed3f(d, -m, m);
    int r = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, r, true);
    return (unsigned)r;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 g_u32x4;
// 16-byte load through a global-address-space pointer (a global_load
// instead of a flat load).
__device__ __forceinline__ uint4 gload16(const void *p)
{
    const u32x4 v = *(g_u32x4 *)(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Network input of Sec. 5.1 at one pixel: [T(r) 3, a 3, (n+1)/2 3, depth 1],
// T(x) = clamp(x,0,1)^(1/gamma) = 2^(log2(x)/gamma), depth scaled to [0,1]
// and clamped.  pack_load only loads the raw values (so that the loads of
// every item are in flight before any result is used); pack_transform maps
// them in place.
__device__ __forceinline__ void pack_load(const FrameDesc &fd, size_t pix, float x[10])
{
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        x[ch] = gload(fd.r + pix * 3 + ch);
        x[3 + ch] = gload(fd.a + pix * 3 + ch);
        x[6 + ch] = gload(fd.n + pix * 3 + ch);
    }
    x[9] = gload(fd.d + pix);
}

__device__ __forceinline__ void pack_transform(const ConvLayer &L, float x[10])
{
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        x[ch] = fast_exp2(fast_log2(fminf(fmaxf(x[ch], 0.f), 1.f)) * L.inv_gamma);
        x[6 + ch] = (x[6 + ch] + 1.f) * 0.5f;
    }
    x[9] = fminf(fmaxf((x[9] - L.dnear) * L.dinv, 0.f), 1.f);
}

// Value held by the neighbouring lane (lane ^ 1), through a DPP quad
// permutation [1, 0, 3, 2] (a VALU move, no LDS round trip).
__device__ __forceinline__ float lane_xor1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));
}

// vmcnt(N) with lgkmcnt(0): waits until at most N vector-memory loads of
// this wave are outstanding (loads complete in order); N = 0 waits for the
// direct-to-LDS loads of the stage.
template <int N>
__device__ __forceinline__ void wait_vmem()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

}  // namespace wskp
