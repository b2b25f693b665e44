// Gathered implicit GEMM on bf16 MFMA behind masked convolutions (3x3 / 1x1,
// stride 2, nearest-2x upsample, two concatenated sources) and the per-token
// linears of the transformer blocks: one argument block.
// launch_igemm gives what is made of 64-channel pieces to wave_gemm.hip (and from
// there 3x3 convolutions of many rows to conv_patch.hip) except compact rows of one
// section from 2048 rows on: those go to linear_wide.hip (float rows, one tile per
// CU) or igemm_dma_kernel; a GroupNorm prologue and 32-channel pieces go to
// igemm_kernel (both igemm.hip).  Products behind a normalisation of 320, 640 or
// 1280 channels have norm_gemm.hip and arguments of their own.  Internal.
#pragma once
#include "common.h"
#include "gemm_choice.h"

namespace fise {

enum { PRO_NONE = 0, PRO_GN = 1, PRO_GN_SILU = 2 };
enum { OUT_COMPACT = 0, OUT_MAP = 1, OUT_TOKENS_T = 2, OUT_COMPACT_F32 = 3 };

// A second destination of a map-producing launch: the consumer's GroupNorm (+SiLU) of the value just stored,
//   dst[pix, c_off + col] = act(x * ss[b, c_off + col].x + ss[b, c_off + col].y),   x = the bf16 value stored at (pix, col)
// with ss the per-(batch element, channel) scale / shift table of that GroupNorm under its CACHED statistics.
// The consumer then reads activations instead of normalising its input in a launch of its own.
struct GnView { bf16_t* dst; const float2* ss; int dstC, c_off, silu, pad_; };

// n / d as (umulhi(n, mul) + n) >> shift: exact for n < 2^31 (round-up method of Granlund and Montgomery)
struct FastDiv { unsigned mul; int shift; };
inline FastDiv fast_div(int d) {
    FastDiv f{1u, 0};
    while ((1ll << f.shift) < d) ++f.shift;
    f.mul = (unsigned)((((unsigned long long)1 << 32) * (((unsigned long long)1 << f.shift) - (unsigned)d)) / (unsigned)d + 1);
    return f;
}

struct IgemmArgs {
    // ---- A operand: rows = B * Ma active pixels (or compact rows) x K
    const bf16_t* a0; const bf16_t* a1; int C0, C1;    // map sources [B,Hin,Win,C*] (a1 unused when C1 == 0)
    int a_compact;                                      // 1: a0 is a compact bf16 [rows, C0] buffer (ksize must be 1)
    int Hin, Win, ksize, stride, ups;
    // ---- row geometry (output map)
    const int* tile_idx; int tile, tile_w, tiles_w, Ho, Wo, B, Ma;   // tiles of tile x tile_w pixels (tile_w 0: square)
    // ---- prologue on A: GroupNorm (+SiLU) with given statistics
    int pro; const float* gn_mean; const float* gn_rstd; const bf16_t* gn_gamma; const bf16_t* gn_beta; int G;
    // ---- B operand: weights [rows_w, K], K innermost
    const bf16_t* w; int N; int K;                      // N = output columns (GEGLU: N = D, weights have 2D rows)
    int geglu;
    // ---- epilogue
    const bf16_t* bias; const float* temb; int temb_stride;
    const bf16_t* res; int res_compact;                 // 0: map at the output pixel, 1: compact bf16 rows, 2: compact float rows
    int nsect, sect_n;                                  // N = nsect * sect_n; section s goes to out[s]
    bf16_t* out[3]; int out_mode[3];
    bf16_t* mirror;                                     // OUT_COMPACT_F32 only: also store a bf16 copy here (may be null)
    // ---- optional LayerNorm of the finished rows (one OUT_COMPACT_F32 section, N = sect_n): ln_out[rows, N] bf16, in a launch of its own.
    const bf16_t* ln_gamma; const bf16_t* ln_beta; float ln_eps; bf16_t* ln_out;
    // ---- optional side product accumulated into the same tile: 1x1 conv of the raw maps s0 | s1
    // [B,Ho,Wo,S*] at the output pixel with weights w2 [N, K2] and bias2 (K2 = S0 + S1, 0 = none)
    const bf16_t* s0; const bf16_t* s1; int S0, S1; const bf16_t* w2; const bf16_t* bias2; int K2;
    // ---- split-K (splits == 1: none)
    int splits; float* partial;
    int gx, gy;                                         // tile grid (row tiles, column tiles); set by the launcher
    int need_pix;                                       // set by the launcher: the epilogue addresses a map (else rows only)
    // ---- optional normalised copies of the output map for its consumers (one OUT_MAP section, N % 4 == 0)
    int nview; GnView view[2];
    // ---- set by the launcher of the wave-split kernel: K steps per workgroup, divisors, arrival counters of split tiles,
    // whether four consecutive rows are four consecutive tokens (8-byte stores into a transposed section)
    // (PATCH: kper chunks of 64 channels and kper2 K steps of the side product)
    int kper, kper2, touch, tt, trans4; int* counters;
    struct { const bf16_t* p; unsigned bytes, pitch; } src[4];      // A sources a0, a1, s0, s1: base, size, bytes per pixel (or row)
    unsigned bias_bytes, bias2_bytes, temb_bytes, res_bytes;        // sizes of the epilogue operands (0: absent)
    FastDiv d_gx, d_gy, d_Ma, d_tt, d_tw, d_tiles_w, d_spt;
};

// What a block of the UNet step keeps in the per-step cache besides its stored maps (all derived from them and from
// the cached statistics): the activated input of its first product (ResNet: SiLU(GN1(x)); transformer: GN(x)), for a
// ResNet also conv2's activated input SiLU(GN2(h1)), the scale / shift tables of those GroupNorms, and the
// normalised copies other blocks want of this block's output.  trust: the derived maps are up to date with the
// stored maps except where this step's producers have just rewritten them (so consumers need not recompute them).
struct BlockDerived {
    void* act_in; void* act_mid; float2* ss_in; float2* ss_mid; int trust;
    GnView out_view[2]; int n_out_view;
};

#if defined(__HIPCC__)
__device__ __forceinline__ unsigned fdiv(unsigned n, FastDiv f) { return (__umulhi(n, f.mul) + n) >> f.shift; }
// A view of a value as stored, before its SiLU: the one expression behind every normalised copy, so that they agree bit for bit.
__device__ __forceinline__ float view_scale(float stored, float scale, float shift) { return fmaf(stored, scale, shift); }
// Four consecutive channels col .. col + 3 of pixel `pix` (batch element b): every view gets its activation.
// In two halves, so that an epilogue can request the table entries of all its items together with its other
// operands and use them later (loaded where they are used, each item pays a round trip of its own in front of
// its stores): view_ss_load fetches the four (scale, shift) pairs per view, put_views4 applies them.
struct ViewSS { float s[2][8]; };
__device__ __forceinline__ void view_ss_load(const GnView* view, int nview, int b, int col, ViewSS& o) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        f32x4_t s01 = {0.f, 0.f, 0.f, 0.f}, s23 = s01;
        if (i < nview) {
            const GnView w = view[i];
            auto sp = (const FISE_AS1 f32x4_t*)(w.ss + (size_t)b * w.dstC + w.c_off + col);
            s01 = sp[0]; s23 = sp[1];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) { o.s[i][q] = s01[q]; o.s[i][4 + q] = s23[q]; }
    }
}
__device__ __forceinline__ void put_views4(const GnView* view, int nview, unsigned pix, int col, const float (&v)[4], const ViewSS& ss) {
    const unsigned p01 = f2bf2(v[0], v[1]), p23 = f2bf2(v[2], v[3]);      // the values as stored
    const float x[4] = {lo16(p01), hi16(p01), lo16(p23), hi16(p23)};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (i >= nview) break;
        const GnView w = view[i];
        float u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = view_scale(x[q], ss.s[i][2 * q], ss.s[i][2 * q + 1]);
        if (w.silu) {
#pragma unroll
            for (int q = 0; q < 4; ++q) u[q] = silu_f(u[q]);
        }
        auto dp = (FISE_AS1 u32x2_t*)(w.dst + (size_t)pix * w.dstC + w.c_off + col);
        *dp = u32x2_t{f2bf2(u[0], u[1]), f2bf2(u[2], u[3])};
    }
}
__device__ __forceinline__ void put_views4(const GnView* view, int nview, int b, unsigned pix, int col, const float (&v)[4]) {
    ViewSS ss;
    view_ss_load(view, nview, b, col, ss);
    put_views4(view, nview, pix, col, v, ss);
}
// One channel (the element-wise epilogue of the register-staged kernel).
__device__ __forceinline__ void put_views1(const GnView* view, int nview, int b, size_t pix, int col, float v) {
    const float x = bf2f(f2bf(v));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (i >= nview) break;
        const GnView w = view[i];
        const float2 s = w.ss[(size_t)b * w.dstC + w.c_off + col];
        float u = view_scale(x, s.x, s.y);
        if (w.silu) u = silu_f(u);
        w.dst[pix * w.dstC + w.c_off + col] = f2bf(u);
    }
}
#endif

struct IgemmWorkspace { float* partial; size_t partial_bytes; int* counters; mutable bool counters_zeroed; };
// One of several products of the same rows: weights [N, K], destination and its OUT_ mode.
struct GemmProduct { const bf16_t* w; int N; bf16_t* out; int mode; };
constexpr int GEMM_GROUP = 32;           // products of one launch
struct GemmGroup { int first[GEMM_GROUP], N[GEMM_GROUP], mode[GEMM_GROUP]; const bf16_t* w[GEMM_GROUP]; bf16_t* out[GEMM_GROUP]; };    // first: column tile where a product starts
// base: compact rows, K and geometry; its weights, width and destinations are the products'.  One launch where the sizes allow it.
int launch_igemm_group(const IgemmArgs& base, const GemmProduct* p, int n, hipStream_t st);
// The same on tiles of up to 224 rows x 112 columns that may straddle products (rows_group.hip).
bool rows_group_takes(const IgemmArgs& base, const GemmProduct* p, int n);
int launch_rows_group(const IgemmArgs& base, const GemmProduct* p, int n, hipStream_t st);
bool wave_gemm_takes(const IgemmArgs& a);
int launch_wave_gemm(IgemmArgs a, const IgemmWorkspace* ws, hipStream_t st);
// 3x3 convolution on tiles of 32 * tm rows x 80 columns (conv_patch.hip; tm 2 or 4, tiles of edge 4 or 8, N a multiple of 80); called with the launcher's fields set.
int launch_conv_patch(const IgemmArgs& a, int tm, hipStream_t st);

// Linears of many compact rows into float rows (linear_wide.hip).
bool linear_wide_takes(const IgemmArgs& a);
int launch_linear_wide(const IgemmArgs& a, hipStream_t st);
#if defined(__HIP_DEVICE_COMPILE__)
// Sum over aligned groups of 16, 32 or 64 lanes, in every lane of the group (data paths of the vector unit: a shuffle through the LDS costs
// ~130 cycles a step, and a row's mean and variance are ten to twelve of them in a row).
template <int CTRL> __device__ __forceinline__ float group_dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int N> __device__ __forceinline__ float group_sum(float x) {
    x += group_dpp<0xB1>(x);                                 // quad_perm 1 0 3 2
    x += group_dpp<0x4E>(x);                                 // quad_perm 2 3 0 1
    x += group_dpp<0x141>(x);                                // row_half_mirror
    x += group_dpp<0x140>(x);                                // row_mirror
    if constexpr (N >= 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    if constexpr (N >= 64) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    return x;
}
// LayerNorm of a row that LPR lanes hold, N pieces of four channels each.
template <int LPR, int N> __device__ __forceinline__ void layer_norm(f32x4_t (&x)[N], const u32x2_t (&gam)[N], const u32x2_t (&bet)[N], float eps) {
    constexpr int C = LPR * N * 4;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) s += (x[j].x + x[j].y) + (x[j].z + x[j].w);
    const float mu = group_sum<LPR>(s) / C;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const f32x4_t d = x[j] - mu;
        q += (d.x * d.x + d.y * d.y) + (d.z * d.z + d.w * d.w);
    }
    const float rs = rsqrtf(group_sum<LPR>(q) / C + eps);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        x[j].x = (x[j].x - mu) * rs * lo16(gam[j].x) + lo16(bet[j].x);
        x[j].y = (x[j].y - mu) * rs * hi16(gam[j].x) + hi16(bet[j].x);
        x[j].z = (x[j].z - mu) * rs * lo16(gam[j].y) + lo16(bet[j].y);
        x[j].w = (x[j].w - mu) * rs * hi16(gam[j].y) + hi16(bet[j].y);
    }
}
// Those pieces as bf16 into row r of an operand in LDS: 16-byte segment p of its 128 bytes at slot p ^ ((r >> 1) & 7).
template <int LPR, int N> __device__ __forceinline__ void put_row(unsigned char* row, int r, int l, const f32x4_t (&x)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int c4 = j * LPR + l, seg = c4 >> 1;       // piece of four channels, 16-byte segment
        *reinterpret_cast<u32x2_t*>(row + (seg >> 3) * 128 + ((seg & 7) ^ ((r >> 1) & 7)) * 16 + (c4 & 1) * 8) = u32x2_t{f2bf2(x[j].x, x[j].y), f2bf2(x[j].z, x[j].w)};
    }
}
#endif

// Normalised rows times weights (norm_gemm.hip).  Rows of K channels: compact float rows under a LayerNorm, or the active pixels of a bf16 map
// [B, Ho*Wo, K] under a LayerNorm, under a GroupNorm with given statistics, or as they are.  N columns in sections of sect_n, section s with
// weights w[s] [sect_n, K] to out[s] (only the last one transposed; geglu: one section, w[0] [2N, K], compact float rows).  A bias belongs to one section, and to a gate or to rows without a
// LayerNorm: the launcher refuses it elsewhere.
enum { NG_ROWS_LN = 0, NG_MAP_LN = 1, NG_MAP_GN = 2, NG_MAP_RAW = 3 };
constexpr bool norm_gemm_has_bias(bool geglu, int src) { return geglu || src == NG_MAP_GN || src == NG_MAP_RAW; }
struct NormGemmArgs {
    const void* x; int src, K;
    const bf16_t* gamma; const bf16_t* beta; float eps;
    const float* gn_mean; const float* gn_rstd; int G;
    const int* tile_idx; int tile, tiles_w, Ho, Wo, B, Ma;
    const bf16_t* w[3]; const bf16_t* bias; int N, sect_n, geglu;
    bf16_t* out[3]; int mode[3];
};
// Cross-attention sub-layer as one launch (cross.hip): out = x + Wo attention(Wq LN(x), K, V) + bias.  tile_idx: x and out are bf16 maps of HW pixels and the
// rows pixels of active tiles; null: compact float rows, which out may be.  Where it and the next one run: cross_form in attention_choice.h.
struct CrossArgs {
    const void* x; void* out; const bf16_t *gamma, *beta, *wq, *wo, *bias, *K, *Vt; float eps;
    int n_ctx, n_stride, B, Ma; const int* tile_idx; int tile, tiles_w, W, HW;
};
int launch_cross(const CrossArgs& a, hipStream_t st);
// The same without the last product and sum, 320 or 640 channels: out = attention(Wq LN(x), K, V), compact bf16 rows.
int launch_query_attention(const CrossArgs& a, int C, hipStream_t st);
bool norm_gemm_takes(int src, int K, int B, int Ma, int H, int W);
int launch_norm_gemm(const NormGemmArgs& a, hipStream_t st);
size_t igemm_workspace_bytes();
// Carves the scratch out of `workspace`; with a null or too
// small workspace `out` is left empty and every launch runs unsplit.
int igemm_workspace_init(void* workspace, size_t bytes, IgemmWorkspace* out, hipStream_t st);
// Enqueue; rows == 0 is a no-op.  `ws` may be null (no split-K).  Returns a fise_status.
int launch_igemm(const IgemmArgs& a, const IgemmWorkspace* ws, hipStream_t st);
// LayerNorm of rows -> compact out[rows, C].  tile_idx == nullptr: `in` is compact [rows, C];
// otherwise `in` is a token map [B, H*W, C] and row r = (b, active pixel r % Ma).
// in_f32 != 0: compact float rows (tile_idx must be nullptr).
int launch_ln_rows(const void* in, int in_f32, int rows, int C, const void* gamma, const void* beta, float eps, void* out,
                   const int* tile_idx, int tile, int tiles_w, int H, int W, int Ma, hipStream_t st);
// views / nview: normalised copies of the output map for its consumers (nullptr / 0 = none)
int conv_dispatch(const fise_conv_args* a, void* workspace, size_t workspace_bytes, hipStream_t st, const GnView* views, int nview);
// out[b, n] = act(bias[n] + sum_k in[b, k] * W[n, k]) for a handful of rows b (float in/out, bf16 weights).
int launch_small_linear(const float* in, int B, int K, const void* W, const void* bias, int N, int silu_out, float* out,
                        hipStream_t st);
int launch_iota(int* p, int n, hipStream_t st);
// ss[B, C] = (rstd * gamma, beta - mean * rstd * gamma): the scale / shift form of a GroupNorm with given statistics.
int launch_gn_scale_shift(const float* mean, const float* rstd, const void* gamma, const void* beta, int B, int C, int G, float2* ss,
                          hipStream_t st);
// act[B,H,W,C0+C1] = GroupNorm(x0|x1) (+SiLU) with the given statistics at the active tiles and their one-pixel ring.
// iw: scratch of the GEMMs that follow on the stream; its arrival counters are zeroed on the way if they are not yet.
int launch_gn_act_halo(const void* x0, const void* x1, int C0, int C1, int B, int H, int W, const float* mean, const float* rstd,
                       const void* gamma, const void* beta, int G, int silu, const int* tile_idx, int n_active, int tile, void* act,
                       hipStream_t st, const IgemmWorkspace* iw = nullptr);
// The same with fresh statistics, in two launches (one for a small map that is active as a whole): those of x0 | x1 to mean / rstd (and the scale / shift table ss [B, C], if given), and act with them
// (workspace as for fise_groupnorm_stats).
int launch_gn_stats_act(const void* x0, const void* x1, int C0, int C1, int B, int H, int W, float eps, float* mean, float* rstd, const void* gamma,
                        const void* beta, int G, int silu, const int* tile_idx, int n_active, int tile, void* act, float2* ss, void* workspace,
                        hipStream_t st, const IgemmWorkspace* iw = nullptr);
// A ResNet block's two activated inputs under given statistics in one launch: act1 as above, of act2 (from h1_cache) the ring only, and the
// scale / shift table ss2 [B, Cout] with which conv1's epilogue writes act2 at the active pixels.
int launch_resnet_acts(const fise_resnet_args* a, void* act1, void* act2, float2* ss2, hipStream_t st, const IgemmWorkspace* iw);
// ws: scratch for the key-split partials (attention_workspace_bytes; null or too small = no key split)
size_t attention_workspace_bytes(int B, int M, int n_keys, int C, int heads);
int launch_attention(const void* q, const void* K, const void* Vt, int B, int M, int n_keys, int n_stride, int C,
                     int heads, float scale, void* out, void* ws, size_t ws_bytes, hipStream_t st);

}  // namespace fise
