// Normalisation kernels: dense GroupNorm statistics (two-stage, deterministic),
// masked GroupNorm+SiLU with given statistics, per-row LayerNorm of compact
// token buffers.
#include <algorithm>
#include <mutex>
#include "conv_choice.h"
#include "igemm.h"

namespace fise {

constexpr int GS_PIX = 64;       // pixels per stage-1 workgroup
constexpr int GS_MAXJ = 4;       // channels per thread per pass (256 threads -> 1024 channels per pass)

// stage 1: partial[b][chunk][g] = (sum, sum of squares) over GS_PIX pixels x the group's channels.
template <typename T>
__global__ __launch_bounds__(256) void gn_partial_kernel(const T* __restrict__ x0, const T* __restrict__ x1, int HW,
                                                         int C0, int C1, int G, double2* __restrict__ partial) {
    extern __shared__ double2 chan[];                    // [C0 + C1]
    const int C = C0 + C1, cpg = C / G;
    const int b = blockIdx.y, chunk = blockIdx.x, nchunk = gridDim.x;
    const int p0 = chunk * GS_PIX, p1 = min(HW, p0 + GS_PIX);
    for (int cbase = 0; cbase < C; cbase += 256 * GS_MAXJ) {
        float s[GS_MAXJ], q[GS_MAXJ];
#pragma unroll
        for (int j = 0; j < GS_MAXJ; ++j) { s[j] = 0.f; q[j] = 0.f; }
        for (int p = p0; p < p1; ++p) {
#pragma unroll
            for (int j = 0; j < GS_MAXJ; ++j) {
                const int c = cbase + threadIdx.x + 256 * j;
                if (c < C) {
                    const float v = c < C0 ? Elem<T>::ld(x0 + ((size_t)b * HW + p) * C0 + c)
                                           : Elem<T>::ld(x1 + ((size_t)b * HW + p) * C1 + (c - C0));
                    s[j] += v; q[j] += v * v;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < GS_MAXJ; ++j) {
            const int c = cbase + threadIdx.x + 256 * j;
            if (c < C) chan[c] = make_double2((double)s[j], (double)q[j]);
        }
    }
    __syncthreads();
    for (int g = threadIdx.x; g < G; g += 256) {
        double s = 0, q = 0;
        for (int c = g * cpg; c < (g + 1) * cpg; ++c) { s += chan[c].x; q += chan[c].y; }
        partial[((size_t)b * nchunk + chunk) * G + g] = make_double2(s, q);
    }
}

// stage 1 for bf16 maps whose channel counts are multiples of 8: 16-byte loads, and the chunk's pixels dealt to as
// many pixel stripes as 256 lanes allow (lane = (stripe, 8-channel piece)), so that a lane's loads do not wait for one
// another.  Stripe sums are float (a dozen terms each), added per channel in stripe order in double.
__global__ __launch_bounds__(256) void gn_partial_vec_kernel(const bf16_t* __restrict__ x0, const bf16_t* __restrict__ x1, int HW,
                                                             int C0, int C1, int G, int gps, double2* __restrict__ partial) {
    extern __shared__ double2 chan[];                    // [channels of the slab], then the stripe sums of one pass
    const int C = C0 + C1, cpg = C / G, tid = threadIdx.x;
    // blockIdx.z: a slab of gps whole groups (its channel range starts and ends on a multiple of 8)
    const int g0 = blockIdx.z * gps, g1 = min(G, g0 + gps);
    const int c_lo = g0 * cpg, CH8 = (g1 - g0) * cpg / 8;
    float2* stripe = reinterpret_cast<float2*>(chan + C);        // [stripes][pieces of the pass][8]
    const int b = blockIdx.y, chunk = blockIdx.x, nchunk = gridDim.x;
    const int p0 = chunk * GS_PIX, p1 = min(HW, p0 + GS_PIX);
    for (int pc = 0; pc < CH8; pc += 256) {
        const int CH = min(256, CH8 - pc), PS = 256 / CH;
        const int cc = tid % CH, ps = tid / CH;
        if (ps < PS) {
            const int c = c_lo + (pc + cc) * 8;
            const bf16_t* src = c < C0 ? x0 + (size_t)b * HW * C0 + c : x1 + (size_t)b * HW * C1 + (c - C0);
            const size_t pitch = c < C0 ? C0 : C1;
            float s[8], q[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) { s[j] = 0.f; q[j] = 0.f; }
#pragma unroll 4                                         // (the loads go out together: one round trip, not one each)
            for (int p = p0 + ps; p < p1; p += PS) {
                const uint4 v = *reinterpret_cast<const uint4*>(src + (size_t)p * pitch);
                const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float lo = lo16(w[j]), hi = hi16(w[j]);
                    s[2 * j] += lo; q[2 * j] += lo * lo; s[2 * j + 1] += hi; q[2 * j + 1] += hi * hi;
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) stripe[(ps * CH + cc) * 8 + j] = make_float2(s[j], q[j]);
        }
        __syncthreads();
        for (int i = tid; i < CH * 8; i += 256) {
            double ds = 0, dq = 0;
#pragma unroll 8
            for (int k = 0; k < PS; ++k) { const float2 v = stripe[k * CH * 8 + i]; ds += (double)v.x; dq += (double)v.y; }
            chan[pc * 8 + i] = make_double2(ds, dq);
        }
        __syncthreads();
    }
    for (int g = g0 + tid; g < g1; g += 256) {
        double s = 0, q = 0;
#pragma unroll 10
        for (int c = g * cpg - c_lo; c < (g + 1) * cpg - c_lo; ++c) { s += chan[c].x; q += chan[c].y; }
        partial[((size_t)b * nchunk + chunk) * G + g] = make_double2(s, q);
    }
}

// stage 2: one wave per (b, g); lane k adds chunks k, k + 64, ... in that order, the 64 lane sums are added in a
// fixed tree.
// With ss the wave also writes the group's channels of the (scale, shift) table, from the rounded statistics it has
// just stored: ss[b, c] = (rstd * gamma[c], beta[c] - mean * rstd * gamma[c]).
__global__ __launch_bounds__(64) void gn_finish_kernel(const double2* __restrict__ partial, int nchunk, int BG, int G, double count,
                                                       float eps, float* __restrict__ mean, float* __restrict__ rstd,
                                                       const bf16_t* __restrict__ gamma, const bf16_t* __restrict__ beta, int C,
                                                       float2* __restrict__ ss) {
    const int i = blockIdx.x, lane = threadIdx.x;
    if (i >= BG) return;
    const int b = i / G, g = i % G;
    double s = 0, q = 0;
    for (int k = lane; k < nchunk; k += 64) { const double2 v = partial[((size_t)b * nchunk + k) * G + g]; s += v.x; q += v.y; }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { s += __shfl_down(s, off); q += __shfl_down(q, off); }
    s = __shfl(s, 0); q = __shfl(q, 0);
    const double m = s / count;
    double var = q / count - m * m;
    if (var < 0) var = 0;
    const float mf = (float)m, rf = (float)(1.0 / sqrt(var + (double)eps));
    if (lane == 0) { mean[i] = mf; rstd[i] = rf; }
    if (ss) {
        const int cpg = C / G;
        for (int c = g * cpg + lane; c < (g + 1) * cpg; c += 64) {
            const float sc = rf * bf2f(gamma[c]);
            ss[(size_t)b * C + c] = make_float2(sc, fmaf(-mf, sc, bf2f(beta[c])));
        }
    }
}

template <typename T>
__global__ void masked_gn_silu_kernel(const T* __restrict__ x, const float* __restrict__ mean, const float* __restrict__ rstd,
                                      const T* __restrict__ gamma, const T* __restrict__ beta, int B, int H, int W, int C,
                                      int G, const int* __restrict__ tile_idx, int Ma, int tile, T* __restrict__ y) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)B * Ma * C;
    if (i >= total) return;
    const int c = (int)(i % C);
    const int m = (int)((i / C) % Ma);
    const int b = (int)(i / ((long long)C * Ma));
    int py, px;
    active_pixel(tile_idx, m, tile, W / tile, py, px);
    const size_t off = (((size_t)b * H + py) * W + px) * C + c;
    const int g = c / (C / G);
    const float u = (Elem<T>::ld(x + off) - mean[b * G + g]) * rstd[b * G + g] * Elem<T>::ld(gamma + c) + Elem<T>::ld(beta + c);
    Elem<T>::st(y + off, silu_f(u));
}

// SiLU(GroupNorm(x)) with given statistics, written once for every pixel of the active tiles AND
// their one-pixel ring (clipped to the image) into a scratch map act[B,H,W,C0+C1]: the 3x3
// convolution that follows reads plain activations instead of re-evaluating the nonlinearity for
// each of its nine taps and each of its column tiles.  Neighbouring tiles write identical values
// to their shared ring.  One thread per (pixel, 8 channels).
// Two maps share a launch: of the second one, whose active pixels the convolution of the first rewrites, only the ring is
// written here (that convolution's epilogue adds its active pixels through the scale / shift table that the launch also writes).
// ResNet block of 1024 rows x 320 channels: two activation launches of 4.5 us -> one of 5.3, the block 27.4 -> 24.5 us; 160 rows, 2560 to
// 1280 channels 56.8 -> 53.7.
struct ActMap {
    const bf16_t* x0; const bf16_t* x1; int C0, C1; const float* mean; const float* rstd; const bf16_t* gamma; const bf16_t* beta; int G, silu;
    bf16_t* act; float2* ss;                             // ss: table to write (null: none)
    int z, cpg; FastDiv d_chunks, d_cpg;                 // workgroups per tile (0: no such map), channels per group; divisors
};

// stat(g): mean and rstd of group g of this workgroup's batch element.
template <bool RING, typename Stat>
__device__ __forceinline__ void act_tile(const ActMap& a, Stat stat, int zi, int H, int W, int t, int tile, FastDiv d_side, FastDiv d_tiles_w) {
    const int b = blockIdx.y, C = a.C0 + a.C1, chunks = C / 8, side = tile + 2, tiles_w = W / tile;
    const int ty = (int)fdiv((unsigned)t, d_tiles_w), y0 = ty * tile - 1, x0 = (t - ty * tiles_w) * tile - 1;
    const int items = (RING ? 4 * (tile + 1) : side * side) * chunks;
    for (int it = zi * 256 + threadIdx.x; it < items; it += a.z * 256) {
        const int p = (int)fdiv((unsigned)it, a.d_chunks), c = (it - p * chunks) * 8;
        int py, px;
        if (RING) {                                      // top row, bottom row, then the two sides
            const int q = p - 2 * side;
            py = q >= 0 ? 1 + (q >> 1) : p >= side ? side - 1 : 0;
            px = q >= 0 ? (q & 1) * (side - 1) : p >= side ? p - side : p;
        } else {
            py = (int)fdiv((unsigned)p, d_side); px = p - py * side;
        }
        const int y = y0 + py, x = x0 + px;
        if (y < 0 || y >= H || x < 0 || x >= W) continue;
        const size_t pix = ((size_t)b * H + y) * W + x;
        const uint4 v = c < a.C0 ? *reinterpret_cast<const uint4*>(a.x0 + pix * a.C0 + c) : *reinterpret_cast<const uint4*>(a.x1 + pix * a.C1 + (c - a.C0));
        const uint4 gv = *reinterpret_cast<const uint4*>(a.gamma + c), bv = *reinterpret_cast<const uint4*>(a.beta + c);
        const unsigned xw[4] = {v.x, v.y, v.z, v.w}, gw[4] = {gv.x, gv.y, gv.z, gv.w}, bw[4] = {bv.x, bv.y, bv.z, bv.w};
        unsigned ow[4];
        // the 8 channels of a chunk lie in one group or straddle one boundary (cpg >= 8 here; else divide per channel)
        const int g0 = (int)fdiv((unsigned)c, a.d_cpg), edge = (g0 + 1) * a.cpg;
        const int g1 = min(g0 + 1, a.G - 1);
        const float2 st0 = stat(g0), st1 = stat(g1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float r[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int cc = c + 2 * e + q;
                float mu, rs;
                if (a.cpg >= 8) { const bool hi = cc >= edge; mu = hi ? st1.x : st0.x; rs = hi ? st1.y : st0.y; }
                else { const float2 sg = stat((int)fdiv((unsigned)cc, a.d_cpg)); mu = sg.x; rs = sg.y; }
                const float xv = q ? hi16(xw[e]) : lo16(xw[e]);
                const float ga = q ? hi16(gw[e]) : lo16(gw[e]);
                const float be = q ? hi16(bw[e]) : lo16(bw[e]);
                const float sc = rs * ga;
                float u = fmaf(xv, sc, fmaf(-mu, sc, be));      // the same two operations as the scale / shift table form
                if (a.silu) u = silu_f(u);
                r[q] = u;
            }
            ow[e] = f2bf2(r[0], r[1]);
        }
        *reinterpret_cast<uint4*>(a.act + pix * C + c) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
    }
}

template <bool PAIR>
__global__ __launch_bounds__(256) void gn_act_halo_kernel(const ActMap first, const ActMap second, int H, int W, const int* __restrict__ tile_idx,
                                                          int tile, FastDiv d_side, FastDiv d_tiles_w, int* __restrict__ zero, int n_zero) {
    const int t = tile_idx[blockIdx.x];
    auto given = [](const ActMap& m) { return [&m](int g) { const int i = blockIdx.y * m.G + g; return make_float2(m.mean[i], m.rstd[i]); }; };
    for (int i = ((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 256 + threadIdx.x; i < n_zero; i += gridDim.x * gridDim.y * gridDim.z * 256) zero[i] = 0;
    if (!PAIR || (int)blockIdx.z < first.z) { act_tile<false>(first, given(first), blockIdx.z, H, W, t, tile, d_side, d_tiles_w); return; }
    const int zi = (int)blockIdx.z - first.z, b = blockIdx.y;
    for (int c = (blockIdx.x * second.z + zi) * 256 + threadIdx.x; c < second.C0; c += gridDim.x * second.z * 256) {
        const int g = (int)fdiv((unsigned)c, second.d_cpg);
        const float sc = second.rstd[b * second.G + g] * bf2f(second.gamma[c]);
        second.ss[b * second.C0 + c] = make_float2(sc, fmaf(-second.mean[b * second.G + g], sc, bf2f(second.beta[c])));
    }
    act_tile<true>(second, given(second), zi, H, W, t, tile, d_side, d_tiles_w);
}

// The same with statistics that are still partial sums (gn_partial_vec_kernel): every workgroup adds up its batch element's chunks, one of them
// stores the statistics and the scale / shift table.  A dense pass with fresh statistics ran a launch of 4.3 us between the two for that (60 of
// them); here it is 32 KB of partial sums (a 64 x 64 map), from L2, in front of the pixels: 5.5 -> 6.6 us.  Whole pass 5377 -> 5207 us.
// 256 / GP lanes a group (GP: the groups, rounded up to a power of two) add every (256 / GP)-th chunk, then one adds the lanes' sums in order.
constexpr int GN_MAX_G = 256;
__global__ __launch_bounds__(256) void gn_finish_act_kernel(const ActMap a, const double2* __restrict__ partial, int nchunk, int log_gp, double count, float eps,
                                                            float* __restrict__ mean, float* __restrict__ rstd, int H, int W, const int* __restrict__ tile_idx, int tile,
                                                            FastDiv d_side, FastDiv d_tiles_w, int* __restrict__ zero, int n_zero) {
    __shared__ double2 sums[256];
    __shared__ float2 stats[GN_MAX_G];
    const int tid = threadIdx.x, b = blockIdx.y, gp = 1 << log_gp, lanes = 256 >> log_gp;
    const int t = tile_idx[blockIdx.x];
    for (int i = ((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 256 + tid; i < n_zero; i += gridDim.x * gridDim.y * gridDim.z * 256) zero[i] = 0;
    {
        const int g = tid & (gp - 1);
        double s = 0, q = 0;
        if (g < a.G) {
            const double2* p = partial + (size_t)b * nchunk * a.G + g;
#pragma unroll 8
            for (int k = tid >> log_gp; k < nchunk; k += lanes) { const double2 v = p[(size_t)k * a.G]; s += v.x; q += v.y; }
        }
        sums[tid] = make_double2(s, q);
    }
    __syncthreads();
    if (tid < a.G) {
        double s = 0, q = 0;
        for (int k = 0; k < lanes; ++k) { const double2 v = sums[(k << log_gp) + tid]; s += v.x; q += v.y; }
        const double m = s / count;
        double var = q / count - m * m;
        if (var < 0) var = 0;
        const float2 st = make_float2((float)m, (float)(1.0 / sqrt(var + (double)eps)));
        stats[tid] = st;
        if (blockIdx.x == 0 && blockIdx.z == 0) { mean[b * a.G + tid] = st.x; rstd[b * a.G + tid] = st.y; }
    }
    __syncthreads();
    const int C = a.C0 + a.C1;
    if (a.ss && blockIdx.x == 0 && blockIdx.z == 0)
        for (int c = tid; c < C; c += 256) {
            const float2 st = stats[fdiv((unsigned)c, a.d_cpg)];
            const float sc = st.y * bf2f(a.gamma[c]);
            a.ss[(size_t)b * C + c] = make_float2(sc, fmaf(-st.x, sc, bf2f(a.beta[c])));
        }
    act_tile<false>(a, [&](int g) { return stats[g]; }, blockIdx.z, H, W, t, tile, d_side, d_tiles_w);
}

// The whole of it as one launch, for small maps of which every pixel is active: a workgroup owns a slab of whole groups (a multiple of 8 channels) over
// all pixels, keeps its values in registers between the sums and the activation, and nothing waits for another workgroup.  A lane holds one piece of eight
// channels of every PS-th pixel; it adds pairs of values in float, the pairs in double.  Bound by its start, one trip to memory and two barriers.
// Two batch elements of 16 x 16 x 1280, sums and activation as two launches and this, us: 4.7 + 5.7 -> 4.9; 2560 channels 8.0.  Dense pass of 64 x 64 4867 -> 4757.
struct GnMapArgs {
    ActMap a; int HW, P, gps, slabs; double count; float eps; float* mean; float* rstd; int* zero; int n_zero;      // P: pieces of a slab, gps: its groups
    FastDiv d_P;
};
template <int J>
__global__ __launch_bounds__(GM_THREADS) void gn_map_kernel(const GnMapArgs g) {
    constexpr int NT = GM_THREADS;
    __shared__ double2 sums[2][NT];
    __shared__ float2 stats[GM_MAX_GROUPS];
    const ActMap& a = g.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.y, C = a.C0 + a.C1;
    for (int i = (b * gridDim.x + blockIdx.x) * NT + tid; i < g.n_zero; i += gridDim.x * gridDim.y * NT) g.zero[i] = 0;
    // neighbouring slabs, which share cache lines, on one XCD
    const int chunk = g.slabs >> 3;
    int w = blockIdx.x;
    if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
    const int ps = (int)fdiv((unsigned)tid, g.d_P), PS = (int)fdiv((unsigned)NT, g.d_P), cc = tid - ps * g.P;
    const int c = w * g.gps * a.cpg + cc * 8;
    const bool live = ps < PS;
    const bf16_t* const src = c < a.C0 ? a.x0 + (size_t)b * g.HW * a.C0 + c : a.x1 + (size_t)b * g.HW * a.C1 + (c - a.C0);
    const size_t pitch = c < a.C0 ? a.C0 : a.C1;
    uint4 v[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = ps + j * PS;
        v[j] = live && p < g.HW ? *reinterpret_cast<const uint4*>(src + (size_t)p * pitch) : make_uint4(0, 0, 0, 0);
    }
    const uint4 gv = *reinterpret_cast<const uint4*>(a.gamma + c), bv = *reinterpret_cast<const uint4*>(a.beta + c);
    // a piece lies in one group or straddles one boundary: its channels from `edge` on belong to the next
    const int gl = (int)fdiv((unsigned)(cc * 8), a.d_cpg), edge = (gl + 1) * a.cpg - cc * 8;
    {
        double2 lo = make_double2(0, 0), hi = make_double2(0, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            double s = 0, q = 0;
#pragma unroll
            for (int j = 0; j < J; j += 2) {
                float x[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const unsigned word = e < 2 ? v[j + k].x : e < 4 ? v[j + k].y : e < 6 ? v[j + k].z : v[j + k].w;
                    x[k] = e & 1 ? hi16(word) : lo16(word);
                }
                s += (double)(x[0] + x[1]); q += (double)(x[0] * x[0] + x[1] * x[1]);
            }
            if (e < edge) { lo.x += s; lo.y += q; } else { hi.x += s; hi.y += q; }
        }
        sums[0][tid] = lo; sums[1][tid] = hi;
    }
    __syncthreads();
    if (wave < g.gps) {
        double s = 0, q = 0;
        for (int i = lane; i < PS * g.P; i += 64) {
            const int r = (int)fdiv((unsigned)i, g.d_P), first = (int)fdiv((unsigned)((i - r * g.P) * 8), a.d_cpg);
            if (first == wave || first + 1 == wave) { const double2 u = sums[first == wave ? 0 : 1][i]; s += u.x; q += u.y; }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) { s += __shfl_xor(s, off); q += __shfl_xor(q, off); }
        const double m = s / g.count;
        double var = q / g.count - m * m;
        if (var < 0) var = 0;
        if (lane == 0) {
            const float2 st = make_float2((float)m, (float)(1.0 / sqrt(var + (double)g.eps)));
            const int i = b * a.G + w * g.gps + wave;
            stats[wave] = st; g.mean[i] = st.x; g.rstd[i] = st.y;
        }
    }
    __syncthreads();
    if (!live) return;
    const float2 st0 = stats[gl], st1 = stats[min(gl + 1, g.gps - 1)];
    const unsigned gw[4] = {gv.x, gv.y, gv.z, gv.w}, bw[4] = {bv.x, bv.y, bv.z, bv.w};
    float sc[8], sh[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float2 st = e < edge ? st0 : st1;
        sc[e] = st.y * (e & 1 ? hi16(gw[e >> 1]) : lo16(gw[e >> 1]));
        sh[e] = fmaf(-st.x, sc[e], e & 1 ? hi16(bw[e >> 1]) : lo16(bw[e >> 1]));
        if (a.ss && ps == 0) a.ss[(size_t)b * C + c + e] = make_float2(sc[e], sh[e]);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = ps + j * PS;
        if (p >= g.HW) break;
        const unsigned xw[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
        unsigned o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float u0 = fmaf(lo16(xw[e]), sc[2 * e], sh[2 * e]), u1 = fmaf(hi16(xw[e]), sc[2 * e + 1], sh[2 * e + 1]);
            if (a.silu) { u0 = silu_f(u0); u1 = silu_f(u1); }
            o[e] = f2bf2(u0, u1);
        }
        *reinterpret_cast<uint4*>(a.act + ((size_t)b * g.HW + p) * C + c) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

__global__ void gn_scale_shift_kernel(const float* __restrict__ mean, const float* __restrict__ rstd, const bf16_t* __restrict__ gamma,
                                      const bf16_t* __restrict__ beta, int B, int C, int G, float2* __restrict__ ss) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B * C) return;
    const int b = i / C, c = i - b * C, g = c / (C / G);
    const float sc = rstd[b * G + g] * bf2f(gamma[c]);
    ss[i] = make_float2(sc, fmaf(-mean[b * G + g], sc, bf2f(beta[c])));
}

int launch_gn_scale_shift(const float* mean, const float* rstd, const void* gamma, const void* beta, int B, int C, int G, float2* ss,
                          hipStream_t st) {
    hipLaunchKernelGGL(gn_scale_shift_kernel, dim3(ceil_div(B * C, 256)), dim3(256), 0, st, mean, rstd, (const bf16_t*)gamma,
                       (const bf16_t*)beta, B, C, G, ss);
    FISE_CHECK_LAUNCH("gn scale/shift table");
    return FISE_OK;
}

static ActMap act_map(const void* x0, const void* x1, int C0, int C1, const float* mean, const float* rstd, const void* gamma, const void* beta, int G,
                      int silu, int tile, bool ring_only, void* act, float2* ss) {
    const int npix = ring_only ? 4 * (tile + 1) : (tile + 2) * (tile + 2), chunks = (C0 + C1) / 8, cpg = (C0 + C1) / G;
    return ActMap{(const bf16_t*)x0, (const bf16_t*)x1, C0, C1, mean, rstd, (const bf16_t*)gamma, (const bf16_t*)beta, G, silu, (bf16_t*)act, ss,
                  std::max(1, std::min(64, ceil_div(npix * chunks, 512))), cpg, fast_div(chunks), fast_div(cpg)};
}

static int launch_act(const ActMap& first, const ActMap* second, int B, int H, int W, const int* tile_idx, int n_active, int tile, hipStream_t st, const IgemmWorkspace* iw) {
    // a launch of its own for the counters costs 2.7 us (a ResNet block of 160 rows x 1280 channels takes 55)
    const bool zero = iw && iw->counters && !iw->counters_zeroed;
    const dim3 grid(n_active, B, first.z + (second ? second->z : 0));
    int* const zp = zero ? iw->counters : nullptr; const int nz = zero ? IGEMM_COUNTERS : 0;
    if (second) hipLaunchKernelGGL(gn_act_halo_kernel<true>, grid, dim3(256), 0, st, first, *second, H, W, tile_idx, tile, fast_div(tile + 2), fast_div(W / tile), zp, nz);
    else hipLaunchKernelGGL(gn_act_halo_kernel<false>, grid, dim3(256), 0, st, first, first, H, W, tile_idx, tile, fast_div(tile + 2), fast_div(W / tile), zp, nz);
    FISE_CHECK_LAUNCH("gn activation with halo");
    if (zero) iw->counters_zeroed = true;
    return FISE_OK;
}

int launch_gn_act_halo(const void* x0, const void* x1, int C0, int C1, int B, int H, int W, const float* mean, const float* rstd,
                       const void* gamma, const void* beta, int G, int silu, const int* tile_idx, int n_active, int tile, void* act,
                       hipStream_t st, const IgemmWorkspace* iw) {
    if (n_active <= 0) return FISE_OK;
    return launch_act(act_map(x0, x1, C0, C1, mean, rstd, gamma, beta, G, silu, tile, false, act, nullptr), nullptr, B, H, W, tile_idx, n_active, tile, st, iw);
}

int launch_resnet_acts(const fise_resnet_args* a, void* act1, void* act2, float2* ss2, hipStream_t st, const IgemmWorkspace* iw) {
    if (a->n_active <= 0) return FISE_OK;
    const ActMap h1 = act_map(a->h1_cache, nullptr, a->Cout, 0, a->gn2_mean, a->gn2_rstd, a->gn2_gamma, a->gn2_beta, a->G, 1, a->tile, true, act2, ss2);
    return launch_act(act_map(a->x0, a->x1, a->C0, a->C1, a->gn1_mean, a->gn1_rstd, a->gn1_gamma, a->gn1_beta, a->G, 1, a->tile, false, act1, nullptr), &h1,
                      a->B, a->H, a->W, a->tile_idx, a->n_active, a->tile, st, iw);
}

// LayerNorm of rows -> compact out[rows, C] (bf16).  General form: one wave per row held in
// registers (C <= 2048): one read, mean, centred variance, one write.  With tile_idx the rows are
// gathered from a token map.
constexpr int LN_MAXJ = 32;
template <typename T>
__global__ __launch_bounds__(256) void ln_rows_kernel(const T* __restrict__ in, int rows, int C,
                                                      const bf16_t* __restrict__ gamma, const bf16_t* __restrict__ beta,
                                                      float eps, bf16_t* __restrict__ out, const int* __restrict__ tile_idx,
                                                      int tile, int tiles_w, int H, int W, int Ma) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    const T* r;
    if (tile_idx) {
        int py, px;
        active_pixel(tile_idx, row % Ma, tile, tiles_w, py, px);
        r = in + (((size_t)(row / Ma) * H + py) * W + px) * C;
    } else {
        r = in + (size_t)row * C;
    }
    float v[LN_MAXJ];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < LN_MAXJ; ++j) {
        const int c = lane + 64 * j;
        v[j] = c < C ? Elem<T>::ld(r + c) : 0.f;
        s += v[j];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    const float mu = s / C;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < LN_MAXJ; ++j) {
        const int c = lane + 64 * j;
        const float d = c < C ? v[j] - mu : 0.f;
        q += d * d;
    }
    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
    const float rs = rsqrtf(q / C + eps);
#pragma unroll
    for (int j = 0; j < LN_MAXJ; ++j) {
        const int c = lane + 64 * j;
        if (c < C) out[(size_t)row * C + c] = f2bf((v[j] - mu) * rs * bf2f(gamma[c]) + bf2f(beta[c]));
    }
}

int launch_ln_rows(const void* in, int in_f32, int rows, int C, const void* gamma, const void* beta, float eps, void* out,
                   const int* tile_idx, int tile, int tiles_w, int H, int W, int Ma, hipStream_t st) {
    if (rows <= 0) return FISE_OK;
    if (C > 64 * LN_MAXJ) return fail(FISE_ERR_SHAPE, "layernorm rows: C=%d > %d", C, 64 * LN_MAXJ);
    const dim3 grid(ceil_div(rows, 4)), block(256);
    if (in_f32)
        hipLaunchKernelGGL(ln_rows_kernel<float>, grid, block, 0, st, (const float*)in, rows, C, (const bf16_t*)gamma,
                           (const bf16_t*)beta, eps, (bf16_t*)out, tile_idx, tile, tiles_w, H, W, Ma);
    else
        hipLaunchKernelGGL(ln_rows_kernel<bf16_t>, grid, block, 0, st, (const bf16_t*)in, rows, C, (const bf16_t*)gamma,
                           (const bf16_t*)beta, eps, (bf16_t*)out, tile_idx, tile, tiles_w, H, W, Ma);
    FISE_CHECK_LAUNCH("layernorm rows");
    return FISE_OK;
}

// A few rows times a weight matrix: one wave per output column, lanes stride over K in
// 8-element (16-byte) weight loads.  K % 8 == 0.
template <int NB>
__global__ __launch_bounds__(256) void small_linear_kernel(const float* __restrict__ in, int K, const bf16_t* __restrict__ W,
                                                           const bf16_t* __restrict__ bias, int N, int silu_out,
                                                           float* __restrict__ out) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (n >= N) return;
    float acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0.f;
    for (int k = lane * 8; k < K; k += 64 * 8) {
        const uint4 wv = *reinterpret_cast<const uint4*>(W + (size_t)n * K + k);
        const unsigned w4[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float wf = (e & 1) ? hi16(w4[e >> 1]) : lo16(w4[e >> 1]);
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = fmaf(in[(size_t)b * K + k + e], wf, acc[b]);
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        float v = acc[b];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) {
            if (bias) v += bf2f(bias[n]);
            out[(size_t)b * N + n] = silu_out ? silu_f(v) : v;
        }
    }
}

int launch_small_linear(const float* in, int B, int K, const void* W, const void* bias, int N, int silu_out, float* out,
                        hipStream_t st) {
    if (K % 8) return fail(FISE_ERR_ALIGN, "small linear: K=%d must be a multiple of 8", K);
    const dim3 grid(ceil_div(N, 4)), block(256);
    for (int b0 = 0; b0 < B; b0 += 2) {
        const float* i0 = in + (size_t)b0 * K; float* o0 = out + (size_t)b0 * N;
        if (B - b0 >= 2)
            hipLaunchKernelGGL(small_linear_kernel<2>, grid, block, 0, st, i0, K, (const bf16_t*)W, (const bf16_t*)bias, N, silu_out, o0);
        else
            hipLaunchKernelGGL(small_linear_kernel<1>, grid, block, 0, st, i0, K, (const bf16_t*)W, (const bf16_t*)bias, N, silu_out, o0);
        FISE_CHECK_LAUNCH("small linear");
    }
    return FISE_OK;
}

__global__ void iota_kernel(int* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i;
}
int launch_iota(int* p, int n, hipStream_t st) {
    if (n <= 0) return FISE_OK;
    hipLaunchKernelGGL(iota_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, p, n);
    FISE_CHECK_LAUNCH("iota");
    return FISE_OK;
}

}  // namespace fise

using namespace fise;

extern "C" size_t fise_groupnorm_stats_workspace_bytes(int B, int H, int W, int C) {
    (void)C;
    if (B < 1 || H < 1 || W < 1) return 0;
    // the group count is not known here: bound it by the channel count
    return align256((size_t)B * ceil_div(H * W, GS_PIX) * (size_t)(C > 0 ? C : 1) * sizeof(double2));
}

// Both entry points below: argument checks, then the two launches with the partial sums in `partial`.
// gamma / beta / ss (all or none): the finish launch also writes the GroupNorm's (scale, shift) table.
static int gn_stats_run(const char* fn, const void* x, const void* x1, int dtype, int B, int H, int W, int C0, int C1, int G,
                        float eps, float* mean, float* rstd, double2* partial, hipStream_t st, const void* gamma = nullptr,
                        const void* beta = nullptr, float2* ss = nullptr, bool finish = true) {
    const int C = C0 + C1;
    const int HW = H * W, nchunk = ceil_div(HW, GS_PIX);
    const size_t shmem = (size_t)C * sizeof(double2);
    constexpr size_t kStripeBytes = 256 * 8 * sizeof(float2);
    if (shmem > 64 * 1024) return fail(FISE_ERR_SHAPE, "%s: C=%d too large", fn, C);
    const bool vec = dtype == FISE_BF16 && C0 % 8 == 0 && C1 % 8 == 0 && shmem + kStripeBytes <= 64 * 1024 && aligned16(x) &&
                     (C1 == 0 || aligned16(x1));
    if (vec) {
        // small maps have few pixel chunks: the groups are dealt to slabs as well (whole groups whose channel range
        // is a multiple of 8 wide), aiming at ~512 workgroups
        const int cpg = C / G;
        const int unit = cpg % 8 == 0 ? 1 : cpg % 4 == 0 ? 2 : cpg % 2 == 0 ? 4 : 8;       // 8 / gcd(cpg, 8) groups
        int gps = G;
        if (G % unit == 0) {
            const int want = std::max(1, 512 / (nchunk * B));
            gps = std::max(unit, ceil_div(ceil_div(G, want), unit) * unit);
        }
        hipLaunchKernelGGL(gn_partial_vec_kernel, dim3(nchunk, B, ceil_div(G, gps)), dim3(256), shmem + kStripeBytes, st, (const bf16_t*)x,
                           (const bf16_t*)x1, HW, C0, C1, G, gps, partial);
    }
    else if (dtype == FISE_F32)
        hipLaunchKernelGGL(gn_partial_kernel<float>, dim3(nchunk, B), dim3(256), shmem, st, (const float*)x, (const float*)x1, HW, C0, C1, G, partial);
    else
        hipLaunchKernelGGL(gn_partial_kernel<bf16_t>, dim3(nchunk, B), dim3(256), shmem, st, (const bf16_t*)x, (const bf16_t*)x1, HW, C0, C1, G, partial);
    FISE_CHECK_LAUNCH("fise_groupnorm_stats(partial)");
    if (!finish) return FISE_OK;
    hipLaunchKernelGGL(gn_finish_kernel, dim3(B * G), dim3(64), 0, st, partial, nchunk, B * G, G,
                       (double)HW * (C / G), eps, mean, rstd, (const bf16_t*)gamma, (const bf16_t*)beta, C, ss);
    FISE_CHECK_LAUNCH("fise_groupnorm_stats(finish)");
    return FISE_OK;
}

static int gn_stats_check(const char* fn, const void* x, const void* x1, int dtype, int B, int H, int W, int C0, int C1, int G,
                          const float* mean, const float* rstd) {
    if (!x || !mean || !rstd) return fail(FISE_ERR_NULL, "%s: null pointer", fn);
    if (dtype != FISE_F32 && dtype != FISE_BF16) return fail(FISE_ERR_DTYPE, "%s: dtype %d", fn, dtype);
    if (C1 < 0 || (C1 > 0 && !x1)) return fail(FISE_ERR_NULL, "%s: second source missing", fn);
    if (B < 1 || H < 1 || W < 1 || C0 < 1 || G < 1 || (C0 + C1) % G) return fail(FISE_ERR_SHAPE, "%s: B%d H%d W%d C%d G%d", fn, B, H, W, C0 + C1, G);
    return FISE_OK;
}

int fise::launch_gn_stats_act(const void* x0, const void* x1, int C0, int C1, int B, int H, int W, float eps, float* mean, float* rstd, const void* gamma,
                              const void* beta, int G, int silu, const int* tile_idx, int n_active, int tile, void* act, float2* ss, void* workspace,
                              hipStream_t st, const IgemmWorkspace* iw) {
    const char* fn = "groupnorm statistics + activation";
    if (!workspace || !gamma || !beta || !act) return fail(FISE_ERR_NULL, "%s: null pointer", fn);
    if (int e = gn_stats_check(fn, x0, x1, FISE_BF16, B, H, W, C0, C1, G, mean, rstd)) return e;
    const int C = C0 + C1;
    if (n_active <= 0 || G > GN_MAX_G) {                 // one after the other
        if (int e = gn_stats_run(fn, x0, x1, FISE_BF16, B, H, W, C0, C1, G, eps, mean, rstd, (double2*)workspace, st, ss ? gamma : nullptr, ss ? beta : nullptr, ss)) return e;
        return launch_gn_act_halo(x0, x1, C0, C1, B, H, W, mean, rstd, gamma, beta, G, silu, tile_idx, n_active, tile, act, st, iw);
    }
    const bool zero = iw && iw->counters && !iw->counters_zeroed;
    const GnSlab slab = gn_slab(C, G);
    const int values = gn_map_values(slab, B, H * W, C, G);
    if ((long long)n_active * tile * tile == (long long)H * W && C0 % 8 == 0 && C1 % 8 == 0 && values && aligned16(x0) && (C1 == 0 || aligned16(x1))) {
        GnMapArgs m{};
        m.a = act_map(x0, x1, C0, C1, mean, rstd, gamma, beta, G, silu, tile, false, act, ss);
        m.HW = H * W; m.P = slab.pieces; m.gps = slab.groups; m.slabs = G / slab.groups; m.count = (double)H * W * (C / G); m.eps = eps; m.mean = mean; m.rstd = rstd;
        m.zero = zero ? iw->counters : nullptr; m.n_zero = zero ? IGEMM_COUNTERS : 0; m.d_P = fast_div(slab.pieces);
        const dim3 grid(m.slabs, B);
        if (values <= 4) hipLaunchKernelGGL(gn_map_kernel<4>, grid, dim3(GM_THREADS), 0, st, m);
        else hipLaunchKernelGGL(gn_map_kernel<GM_MAX_J>, grid, dim3(GM_THREADS), 0, st, m);
        FISE_CHECK_LAUNCH("gn statistics and activation of a map");
        if (zero) iw->counters_zeroed = true;
        return FISE_OK;
    }
    if (int e = gn_stats_run(fn, x0, x1, FISE_BF16, B, H, W, C0, C1, G, eps, mean, rstd, (double2*)workspace, st, nullptr, nullptr, nullptr, false)) return e;
    ActMap a = act_map(x0, x1, C0, C1, mean, rstd, gamma, beta, G, silu, tile, false, act, ss);
    a.z = std::max(1, std::min(a.z, 1024 / (n_active * B)));      // each workgroup reads the partial sums: four to a CU at most
    int log_gp = 0;
    while ((1 << log_gp) < G) ++log_gp;
    hipLaunchKernelGGL(gn_finish_act_kernel, dim3(n_active, B, a.z), dim3(256), 0, st, a, (const double2*)workspace, ceil_div(H * W, GS_PIX), log_gp,
                       (double)H * W * (C / G), eps, mean, rstd, H, W, tile_idx, tile, fast_div(tile + 2), fast_div(W / tile), zero ? iw->counters : nullptr,
                       zero ? IGEMM_COUNTERS : 0);
    FISE_CHECK_LAUNCH("gn statistics and activation with halo");
    if (zero) iw->counters_zeroed = true;
    return FISE_OK;
}

extern "C" int fise_groupnorm_stats(const void* x, const void* x1, int dtype, int B, int H, int W, int C0, int C1, int G,
                                    float eps, float* mean, float* rstd, void* workspace, void* stream) {
    const char* fn = "fise_groupnorm_stats";
    if (!workspace) return fail(FISE_ERR_NULL, "%s: null pointer", fn);
    if (int e = gn_stats_check(fn, x, x1, dtype, B, H, W, C0, C1, G, mean, rstd)) return e;
    return gn_stats_run(fn, x, x1, dtype, B, H, W, C0, C1, G, eps, mean, rstd, (double2*)workspace, as_stream(stream));
}

// ---- the same statistics for callers that can pass no workspace: the per-chunk partial sums live in a fixed array
// in device memory that belongs to the library (one copy per GPU, held until the process ends).
constexpr size_t GN_STATIC_BYTES = 1u << 20;                      // 65536 (batch element, chunk, group) partial sums
static __device__ __align__(256) unsigned char scratch[GN_STATIC_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];                                 // device address of `scratch` on each GPU (null: not asked yet)

// Device address of this GPU's copy of `scratch`.  In host code the array's name is only a handle: the address a
// kernel can use comes from hipGetSymbolAddress, asked once per device with that device current.
int static_scratch(const char* fn, void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return fail(FISE_ERR_HIP, "%s: no current device", fn);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail(FISE_ERR_HIP, "%s: hipGetSymbolAddress: %s", fn, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return FISE_OK;
}
}  // namespace

extern "C" size_t fise_groupnorm_stats_static_capacity_bytes(void) { return GN_STATIC_BYTES; }

extern "C" int fise_groupnorm_stats_static(const void* x, const void* x1, int dtype, int B, int H, int W, int C0, int C1, int G,
                                           float eps, float* mean, float* rstd, void* stream) {
    const char* fn = "fise_groupnorm_stats_static";
    if (int e = gn_stats_check(fn, x, x1, dtype, B, H, W, C0, C1, G, mean, rstd)) return e;
    const size_t need = (size_t)B * ceil_div(H * W, GS_PIX) * (size_t)G * sizeof(double2);
    if (need > GN_STATIC_BYTES)
        return fail(FISE_ERR_CAPACITY, "%s: B=%d x %d chunks of %d pixels x G=%d partial sums need %zu bytes, the fixed scratch holds %zu",
                    fn, B, ceil_div(H * W, GS_PIX), GS_PIX, G, need, (size_t)GN_STATIC_BYTES);
    void* partial = nullptr;
    if (int e = static_scratch(fn, &partial)) return e;
    // every partial sum the second launch reads is written by the first: nothing has to start at zero
    return gn_stats_run(fn, x, x1, dtype, B, H, W, C0, C1, G, eps, mean, rstd, (double2*)partial, as_stream(stream));
}

extern "C" int fise_masked_groupnorm_silu(const void* x, const float* mean, const float* rstd, const void* gamma,
                                          const void* beta, int dtype, int B, int H, int W, int C, int G,
                                          const int32_t* tile_idx, int n_active, int tile, void* y_cache, void* stream) {
    if (!x || !mean || !rstd || !gamma || !beta || !y_cache) return fail(FISE_ERR_NULL, "fise_masked_groupnorm_silu: null pointer");
    if (dtype != FISE_F32 && dtype != FISE_BF16) return fail(FISE_ERR_DTYPE, "fise_masked_groupnorm_silu: dtype %d", dtype);
    if (B < 1 || H < 1 || W < 1 || C < 1 || G < 1 || C % G || tile < 1 || H % tile || W % tile)
        return fail(FISE_ERR_SHAPE, "fise_masked_groupnorm_silu: B%d H%d W%d C%d G%d tile%d", B, H, W, C, G, tile);
    if (n_active < 0 || n_active > (H / tile) * (W / tile)) return fail(FISE_ERR_CAPACITY, "fise_masked_groupnorm_silu: n_active %d", n_active);
    if (n_active == 0) return FISE_OK;
    if (!tile_idx) return fail(FISE_ERR_NULL, "fise_masked_groupnorm_silu: null tile_idx");
    const int Ma = n_active * tile * tile;
    const long long total = (long long)B * Ma * C;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (dtype == FISE_F32)
        hipLaunchKernelGGL(masked_gn_silu_kernel<float>, grid, block, 0, as_stream(stream), (const float*)x, mean, rstd,
                           (const float*)gamma, (const float*)beta, B, H, W, C, G, tile_idx, Ma, tile, (float*)y_cache);
    else
        hipLaunchKernelGGL(masked_gn_silu_kernel<bf16_t>, grid, block, 0, as_stream(stream), (const bf16_t*)x, mean, rstd,
                           (const bf16_t*)gamma, (const bf16_t*)beta, B, H, W, C, G, tile_idx, Ma, tile, (bf16_t*)y_cache);
    FISE_CHECK_LAUNCH("fise_masked_groupnorm_silu");
    return FISE_OK;
}
