// Internal declarations shared by the HIP kernels and the C ABI layer of
// libwskp.  Not part of the public interface (include/wskp.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace wskp {

constexpr int kMaxLevels = 6;
constexpr int kMaxKernels = 8;
constexpr int kThreads = 256;  // every kernel runs 4 wave64s per workgroup

// Everything one frame's layers need: its size, the caller's input and
// output buffers, and where its intermediate maps sit in the workspace.
struct FrameDesc {
    int H, W;
    const float *r, *a, *n, *d;  // radiance, albedo, normal [H,W,3]; depth [H,W,1]
    float *out;                  // [H,W,3]
    void *e[kMaxLevels];         // encoder outputs e_l  [H>>l, W>>l, C_l]
    void *u[kMaxLevels];         // decoder outputs u_l  [H>>l, W>>l, C_l]; u[L-1] == e[L-1]
    void *p[kMaxLevels];         // bf16 form: 2x2 means of e_l [H>>(l+1), W>>(l+1), C_l]
    float *head;                 // [H,W,2M]: weights W_i then logits
};

// Global-memory access through address-space-1 pointers.  Pointers that
// reach a kernel inside a structure are generic, and generic (flat)
// accesses also count against the LDS wait counter: every wait for an LDS
// read would then also wait for the global loads still in flight.
template <typename T>
__device__ __forceinline__ T gload(const T *p)
{
    return *(const __attribute__((address_space(1))) T *)p;
}
template <typename T>
__device__ __forceinline__ void gstore(T *p, T v)
{
    *(__attribute__((address_space(1))) T *)p = v;
}
// N consecutive floats from an address of any float alignment, in the widest
// loads that N allows (the hardware takes them at 4-byte alignment, which the
// types state: gload and gstore would deduce the types' natural alignment).
typedef float uf4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float uf2 __attribute__((ext_vector_type(2), aligned(4)));
template <int N>
__device__ __forceinline__ void load_floats(const float *p, float *v)
{
    if constexpr (N >= 4) {
        const uf4 q = *(const __attribute__((address_space(1))) uf4 *)p;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = q[i];
        if constexpr (N > 4) load_floats<N - 4>(p + 4, v + 4);
    } else if constexpr (N >= 2) {
        const uf2 q = *(const __attribute__((address_space(1))) uf2 *)p;
        v[0] = q[0];
        v[1] = q[1];
        if constexpr (N > 2) load_floats<N - 2>(p + 2, v + 2);
    } else if constexpr (N == 1) {
        v[0] = gload(p);
    }
}
template <int N>
__device__ __forceinline__ void store_floats(float *p, const float *v)
{
    if constexpr (N >= 4) {
        *(__attribute__((address_space(1))) uf4 *)p = uf4{v[0], v[1], v[2], v[3]};
        if constexpr (N > 4) store_floats<N - 4>(p + 4, v + 4);
    } else if constexpr (N >= 2) {
        *(__attribute__((address_space(1))) uf2 *)p = uf2{v[0], v[1]};
        if constexpr (N > 2) store_floats<N - 2>(p + 2, v + 2);
    } else if constexpr (N == 1) {
        gstore(p, v[0]);
    }
}

typedef float gf32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int gu32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int gu32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier without the memory fence of __syncthreads(): the fence
// waits for every global load in flight (prefetches included).  Callers make
// the data they need visible explicitly (wait_lds / a vmcnt wait before the
// barrier); the empty asm statements keep the compiler from moving memory
// accesses across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// lgkmcnt(0): this wave's LDS reads and writes have completed.
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt((15) | (3 << 14) | (7 << 4) | (0 << 8)); }

// Barrier for LDS producer/consumer phases: this wave's LDS accesses are
// complete, then every wave of the workgroup has arrived.  Global loads
// stay in flight.
__device__ __forceinline__ void lds_sync()
{
    wait_lds();
    lds_barrier();
}

// A batch of frames for one launch: either one frame passed by value or a
// device-resident table of n frames.
struct FrameArg {
    const FrameDesc *table;  // device pointer, or nullptr to use `one`
    int first, n;            // the launch covers frames first .. first + n - 1 of the table
    int reverse;             // walk tiles in reverse order
    // capacity launch (graph replay): when non-null, dev_n[0] and dev_n[1] are
    // first and n and dev_n[2 + launch] is this launch's tile count, all in
    // device memory, and the grid is an upper bound on those tiles;
    // workgroups beyond them exit
    const int *dev_n;
    int launch;
    FrameDesc one;
};

__device__ __forceinline__ const FrameDesc &frame_at(const FrameArg &fa, int f)
{
    return fa.table ? fa.table[f] : fa.one;
}

// Raw buffer resource over `bytes` bytes at `base`.  Loads through it
// whose offset lies beyond `bytes` return zeros.  The descriptor must live
// in scalar registers: base and size are made visibly wave-uniform (the
// callers pass wave-uniform values).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void *base, unsigned bytes)
{
    const unsigned long long b = reinterpret_cast<unsigned long long>(base);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    void *ub = reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, (int)__builtin_amdgcn_readfirstlane(bytes),
                                             0x00020000);
}

// Spread consecutive logical tile ids over one XCD.  The hardware deals
// workgroups round-robin to the 8 XCDs (block b runs on XCD b % 8); this
// bijection gives each XCD a contiguous run of logical ids so that tiles
// that share halos (and output-channel groups that share an input tile)
// share that XCD's L2.
__device__ __forceinline__ int xcd_logical_id(int b, int nb)
{
    const int x = b & 7, i = b >> 3;
    const int q = nb >> 3, rmd = nb & 7;
    return x * q + (x < rmd ? x : rmd) + i;
}

// Finds the frame of a batch that holds logical tile t, given the tile
// count of a frame of size H x W, and rewrites t as the tile index inside
// that frame.  Each lane reads one frame's size, a wave-wide inclusive scan
// turns the counts into cumulative ends, and a ballot counts the frames
// that end at or before t: one round of loads per 64 frames instead of one
// dependent load per frame.  Returns -1 past the batch's last tile.  Every
// lane of the wave calls it with the same t; the results are wave-uniform.
// The frames are first .. first + n - 1 of the table.
template <typename Count>
__device__ __forceinline__ int batch_frame(const FrameArg &fa, int first, int n, int &t, Count count)
{
    if (!fa.table) return t < count(fa.one.H, fa.one.W) ? 0 : -1;
    const int lane = threadIdx.x & 63;
    int base = 0;
    for (int f0 = 0; f0 < n; f0 += 64) {
        const int f = f0 + lane;
        int c = f < n ? count(gload(&fa.table[first + f].H), gload(&fa.table[first + f].W)) : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(c, d, 64);
            if (lane >= d) c += v;
        }
        const int end = base + c;
        const int k = __popcll(__ballot(f < n && end <= t));
        const int valid = n - f0 < 64 ? n - f0 : 64;
        if (k < valid) {
            t = __builtin_amdgcn_readfirstlane(t - (k > 0 ? __shfl(end, k - 1, 64) : base));
            return __builtin_amdgcn_readfirstlane(first + f0 + k);
        }
        base = __shfl(end, 63, 64);
    }
    return -1;
}

// Logical tile of workgroup b of a launch of nb workgroups, and the frames
// first .. first + n - 1 it covers.  Capacity launches read these and the
// launch's tile count from device memory (one load round: the words share a
// cache line); there the tile count is below nb, and workgroups beyond it
// get -1.  Then the XCD-aware spread of the ids over the real tile count and
// the optional reversal.
__device__ __forceinline__ int batch_tile_id(const FrameArg &fa, int b, int nb, int &first, int &n)
{
    first = fa.first;
    n = fa.n;
    if (fa.dev_n) {
        const int df = gload(fa.dev_n), dn = gload(fa.dev_n + 1), dt = gload(fa.dev_n + 2 + fa.launch);
        first = __builtin_amdgcn_readfirstlane(df);
        n = __builtin_amdgcn_readfirstlane(dn);
        nb = __builtin_amdgcn_readfirstlane(dt);
        if (b >= nb) return -1;
    }
    int t = xcd_logical_id(b, nb);
    if (fa.reverse) t = nb - 1 - t;
    return t;
}


enum ConvMode { CONV_PACK = 0, CONV_POOL = 1, CONV_CAT = 2, CONV_PLAIN = 3 };
// EPI_BWD_*: the input gradient of a conv in training (conv_split.hip).
enum ConvEpi { EPI_RELU = 0, EPI_HEAD_SOFTPLUS = 1, EPI_HEAD_EXP = 2, EPI_BWD_MASK = 3, EPI_BWD_CAT = 4, EPI_BWD_POOL = 5 };
enum ActType { ACT_F32 = 0, ACT_BF16 = 1 };

// One 3x3 conv layer as the kernels see it.
struct ConvLayer {
    int level;         // output resolution level (H >> level, W >> level)
    int src0_kind;     // 0: e[src0_idx], 1: u[src0_idx], 2: p[src0_idx]
    int src0_idx;
    int src1_idx;      // CAT: skip e[src1_idx]
    int C0, C1;        // channels of source 0 / source 1 (CAT: up, skip)
    int Cin_pad;       // virtual input channels padded to the chunk size
    int Cout;          // real output channels
    int Cout_pad;      // padded to 16 * NB * groups
    int groups;        // output-channel groups (one workgroup each)
    int out_kind;      // 0: e[out_idx], 1: u[out_idx], 2: head
    int out_idx;
    int M;             // head: channels 0..M-1 get the weight activation
    int CK;            // input channels per reduction chunk (weights packed to match)
    int NB;            // 16-channel output blocks per workgroup
    int th;            // output rows per tile of the kernel that runs this layer (TH of its template)
    int ks;            // kernel size: 3, or 5 (a merged RepVGG block)
    int pool_idx;      // >= 0: the epilogue also writes the 2x2 means of the output to p[pool_idx]
    const void *w;     // packed weights
    const float *bias; // [Cout]
    float inv_gamma, dnear, dinv;  // CONV_PACK preprocessing constants
    float in_qscale;           // fp8: 1 / (input activation scale)
    const float *out_scale;    // fp8: per output channel, input scale x weight scale
};

struct DecodeCfg {
    int M;
    int R;                    // max radius
    int radius[kMaxKernels];  // (k_i - 1)/2
    float eps_norm;
    float eps_albedo;
    int exp_weights;          // frames form: the head holds h, W = exp(h) (per-tile shift)
    int tw, th;               // forward decode tile: centres per row, rows
    int hxs;                  // row stride (float4) of its LDS plane
};

// ---- launchers (defined in the .hip files) --------------------------------
// Launches one conv layer over `blocks` workgroups (conv_grid of the batch;
// a larger count is allowed: surplus workgroups exit at once).
hipError_t launch_conv(const ConvLayer &L, int mode, int epi, int prec, const FrameArg &fa,
                       int blocks, hipStream_t s);
int conv_grid(const ConvLayer &L, int n, const int *H, const int *W);
// fp32 native convs: sets the layer's tiling for these sizes, returns its grid
int conv_fp32_tiles(ConvLayer &L, int n, const int *H, const int *W);
// fp8 convs: tile rows for these sizes
int conv_fp8_rows(const ConvLayer &L, int mode, int n, const int *H, const int *W);
// FP32 3x3 convs on the bf16 matrix cores (conv_split.hip): sets the layer's
// tiling for Cin input channels (Cout set), sizes its packed weights, launches
// it.
void conv_split_layer(ConvLayer &L, int Cin);
size_t conv_split_weight_bytes(int Cin, int Cout);
// fp32 weights packed on the device, every layer in one launch
enum PackKind { PACK_SPLIT = 0, PACK_SPLIT_DGRAD = 1, PACK_NATIVE = 2 };
struct PackJob {
    int kind, Ci, Co, nch, groups, CK, Cout_pad, block0;
    const float *w;
    void *out;
    float *bias;
};
constexpr int kMaxPackJobs = 4 * kMaxLevels;   // both layouts of 2 levels - 1 convs and the head
struct PackJobs {
    int n = 0, blocks = 0;
    PackJob j[kMaxPackJobs];
    void add_split(int Ci, int Co, bool dgrad, const float *w, void *out);
    void add_native(int Ci, int Co, int CK, int nch, int Cout_pad, const float *w, float *out, float *bias);
};
hipError_t launch_conv_pack(const PackJobs &jobs, hipStream_t s);
hipError_t launch_conv_split(const ConvLayer &L, int mode, int epi, const FrameArg &fa, int blocks, hipStream_t s);
int conv_chunk(int prec, int mode, int Cin, int C0);
// 16-channel output blocks per workgroup for a layer with nblk blocks.
int conv_blocks_per_group(int prec, int mode, int CK, int nblk, int ks);
// bf16 layers of conv_bf16.hip: tile rows for n frames, and the launch
int conv_bf16_rows(const ConvLayer &L, int n, const int *H, const int *W);
hipError_t launch_conv_bf16(const ConvLayer &L, int mode, const FrameArg &fa, int blocks, hipStream_t s);
// Decode + fusion + remodulation over frames of fa (denoise mode: c and mod
// derive from r, a) -- or over plain tensors (decode mode).
hipError_t launch_decode_frames(const DecodeCfg &dc, const FrameArg &fa, int blocks, hipStream_t s);
// Sets dc.tw, dc.th, dc.hxs from dc.R (the forward decode's tile shape).
void decode_tile_shape(DecodeCfg &dc);
int decode_grid(const DecodeCfg &dc, int n, const int *H, const int *W);
// the forward decode's tile for a batch of these sizes
DecodeCfg decode_frames_cfg(const DecodeCfg &dc, int n, const int *H, const int *W);
hipError_t launch_decode_tensors(const DecodeCfg &dc, int N, int H, int W, const float *head,
                                 const float *c, const float *mod, float *out, hipStream_t s);
// wskp_decode of 1..kMrJoint levels of one frame in one launch, level l's irradiance
// the l times pooled c, no remodulation
constexpr int kMrJoint = 3;
hipError_t launch_decode_levels(const DecodeCfg &dc, int levels, int H, int W, const float *const *heads,
                                const float *c, float *const *outs, hipStream_t s);
// act_ld > 0 (training): grad_head receives the gradient of the head conv's
// output instead, rows of act_ld >= 2M floats: the weights' part times
// softplus' (= -expm1(-W)), the logits', zeros; grad_c is not written.
hipError_t launch_decode_backward(const DecodeCfg &dc, int N, int H, int W, const float *head,
                                  const float *c, const float *mod, const float *g,
                                  float *grad_head, float *grad_c, void *scratch, int act_ld,
                                  hipStream_t s);
size_t decode_backward_scratch_bytes(const DecodeCfg &dc, int N, int H, int W);
// Training kernels (train.hip): see the file's header for each operation.
// Kernels with an nf argument run over nf frames of one size: frame f's
// operand X is at X + f sX (strides in floats); their outputs are contiguous
// per frame.
// Up to kTrGroup frames' own buffers (radiance, albedo, normal, depth, the
// denoised output, the reference) for the per-frame training kernels, which
// run over the frames of a group in one launch
constexpr int kTrGroup = 16;
struct TrFrames {
    const float *r[kTrGroup], *a[kTrGroup], *n[kTrGroup], *d[kTrGroup], *y[kTrGroup], *t[kTrGroup];
};
hipError_t tr_pack(long P, int nf, const TrFrames &fr, float inv_gamma, float dnear, float dinv, float *X,
                   hipStream_t s);
hipError_t tr_pool(int H, int W, int C, int nf, const float *in, long sin, float *out, hipStream_t s);
hipError_t tr_head_prep(long P, int M, int nf, const float *planar, long sp, const TrFrames &fr, float eps_a,
                        float *head, float *c, float *mod, hipStream_t s);
int tr_smape_blocks(long n);
// loss[0] (+)= the SMAPE of nf frames of n values (partial: nf x
// tr_smape_blocks(n) floats)
hipError_t tr_smape(long n, int nf, const TrFrames &fr, float eps, float inv_n, float *g, float *partial, float *loss,
                    int accumulate, hipStream_t s);
// partial sums of a weight gradient over nf frames
size_t tr_wgrad_part_floats(int H, int W, int Ci, int Co, int nf);
// its kernel (train_wgrad.hip) and the number of partial sums it writes
int tr_wgrad_strips(int H, int W, int Ci, int Co, int nf);
hipError_t launch_wgrad_split(int H, int W, int Co, int ldg, int nf, const float *gm, long sgm, const float *in,
                              long sin, int Cf, const float *up, long sup, int Cu, float *part, float *partb,
                              hipStream_t s);
// The conv's input: Cu channels of `up` (H/2 x W/2) upsampled x2, then Cf
// channels of `in` (H x W) (Cu = 0: `in` alone); gm rows are ldg >= Co
// floats apart; dw and db receive the sum of the nf frames, added to what is
// there if accumulate
hipError_t tr_wgrad(int H, int W, int Co, int ldg, int nf, const float *gm, long sgm, const float *in, long sin,
                    int Cf, const float *up, long sup, int Cu, float *part, float *dw, float *db, bool accumulate,
                    hipStream_t s);
// Tables of nf frames for the input-gradient convs, all in one launch: table k's
// descriptors at tab + k nf, of H x W with e[0] = src, e[1] = dst, e[2] = dst2,
// u[0] = act of the frame (frame strides in floats).
struct TrConvFrames {
    int H, W;
    const float *src, *act;
    float *dst, *dst2;
    long ss, sa, sd, sd2;
};
struct TrConvTables {
    int n = 0;
    TrConvFrames t[2 * kMaxLevels];
};
__host__ __device__ inline FrameDesc tr_conv_frame(const TrConvFrames &t, int f)
{
    FrameDesc d{};
    d.H = t.H;
    d.W = t.W;
    d.e[0] = const_cast<float *>(t.src + f * t.ss);
    d.e[1] = t.dst + f * t.sd;
    d.e[2] = t.dst2 ? t.dst2 + f * t.sd2 : nullptr;
    d.u[0] = t.act ? const_cast<float *>(t.act + f * t.sa) : nullptr;
    return d;
}
hipError_t tr_frame_tables(FrameDesc *tab, int nf, const TrConvTables &tables, hipStream_t s);
hipError_t tr_adam(long n, float *w, const float *g, float *m, float *v, float lr, float b1, float b2, float c1,
                   float c2, float eps, hipStream_t s);
// Multi-resolution reconstruction pieces (mr.hip): 2x2 mean of a 3-channel
// image, and the Eq. 7 blend (optionally remodulated).
hipError_t launch_pool2(int H, int W, const float *in, float *out, hipStream_t s);
// Every blend of L levels (2..6) in one launch: f[l] the filtered images,
// alpha[l] (l < L - 1) their weights.
hipError_t launch_mr_blend_all(int L, int H, int W, const float *const *f, const float *const *alpha,
                               const float *mod, float *out, hipStream_t s);
hipError_t launch_mr_blend(int H, int W, const float *fine, const float *coarse, const float *alpha,
                           const float *mod, float *out, hipStream_t s);
// Temporal accumulation of one frame (temporal.hip); pr == nullptr: first frame.
hipError_t launch_temporal(int H, int W, const float *r, const float *n, const float *wp, const float *mv,
                           const float *pr, const float *pl, const float *pn, const float *pw, float alpha_min,
                           float pos_tol, float normal_tol, float *out, float *len, hipStream_t s);
// Explicit kernel-map reconstruction (the comparison of Sec. 5.3, kp.hip).
size_t kp_map_floats(const DecodeCfg &dc, int H, int W);
hipError_t launch_kp_expand(const DecodeCfg &dc, int H, int W, const float *head, float *maps, hipStream_t s);
hipError_t launch_kp_decode(const DecodeCfg &dc, int H, int W, const float *maps, const float *head,
                            const float *c, const float *mod, float *out, hipStream_t s);

// Tile geometry of the conv kernels (host and device agree on these).
constexpr int kConvTW = 32;  // output columns per tile (two 16-pixel MFMA blocks)
int conv_tile_rows(int prec, int mode, int CK, int level, bool pool, int ks);
// true if the layer runs the direct-to-LDS bf16 kernel (its weights are
// packed without row padding and with swizzled column groups)
bool conv_uses_direct(int prec, int mode, int CK, int ks);

}  // namespace wskp
