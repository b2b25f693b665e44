// Mask generation kernels: per-pixel difference + threshold, tile OR-reduce with
// ordered compaction (wave ballot + popcount prefix), 2x2 OR-pool, multi-step
// difference accumulation, Otsu threshold search, block counts for the
// adaptive block-size choice.
#include <algorithm>
#include "common.h"
#include "ordered_sum.h"

namespace fise {

// ---------------------------------------------------------------------------
// d = mean_{b,c} |fresh - cached| with a fixed summation order (b outermost, c ascending, float adds), one pixel per lane.
//  - slab form: the workgroup stages [PIX pixels x DET_CH channels] through LDS so that global reads are coalesced along channels
//    while each pixel's channels are still added in ascending order by one lane.  Bound by the round trip of the loads and the chain of
//    additions; maps of few pixels are cut into groups of 16 to reach more CUs (32 x 32 x 64 fp32: 6.7 -> 3.3 us).
//  - vector form (4, 8, 12 or 16 channels, which a lane reads as vectors of four): no LDS, every load of two batch elements in
//    flight at once (64 x 64 x 4 bf16, batch 2: 4.0 -> 2.4 us).
// ---------------------------------------------------------------------------
constexpr int DET_CH = 64;          // channels staged per slab
constexpr int DET_THREADS = 256;    // all four waves load the slab; the first sums it, one pixel per lane

__device__ __forceinline__ void pixel_put(float s, int p, int terms, float* __restrict__ d_out, int accumulate, float threshold,
                                          uint8_t* __restrict__ pix) {
    const float d = s / (float)terms;
    if (d_out) d_out[p] = accumulate ? d_out[p] + d : d;
    if (pix) pix[p] = d > threshold ? 1 : 0;
}

template <typename T, int DET_PIX>
__global__ __launch_bounds__(DET_THREADS) void pixel_diff_kernel(const T* __restrict__ cached, const T* __restrict__ fresh,
                                                                 int B, int HW, int C, float* __restrict__ d_out,
                                                                 int accumulate, float threshold, uint8_t* __restrict__ pix) {
    __shared__ __attribute__((aligned(16))) float slab[DET_PIX][DET_CH + 4];
    const int p0 = blockIdx.x * DET_PIX;
    const int tid = threadIdx.x;
    float s = 0.f;
    auto absdiff = [&](int b, int pp, int c) {
        const int p = p0 + pp;
        if (p >= HW) return 0.f;
        const size_t off = ((size_t)b * HW + p) * C + c;
        return fabsf(Elem<T>::ld(fresh + off) - Elem<T>::ld(cached + off));
    };
    for (int b = 0; b < B; ++b) {
        for (int c0 = 0; c0 < C; c0 += DET_CH) {
            const int nc = min(DET_CH, C - c0);
            // cooperative load: consecutive lanes walk channels of one pixel, then the next pixel
            if (nc == DET_CH) {                 // full slab: constant trip count, all loads of a lane in flight together
                float v[DET_PIX * DET_CH / DET_THREADS];
#pragma unroll
                for (int j = 0; j < DET_PIX * DET_CH / DET_THREADS; ++j) {
                    const int e = tid + j * DET_THREADS;
                    v[j] = absdiff(b, e / DET_CH, c0 + e % DET_CH);
                }
#pragma unroll
                for (int j = 0; j < DET_PIX * DET_CH / DET_THREADS; ++j) {
                    const int e = tid + j * DET_THREADS;
                    slab[e / DET_CH][e % DET_CH] = v[j];
                }
            } else {
                for (int e = tid; e < DET_PIX * nc; e += DET_THREADS) slab[e / nc][e % nc] = absdiff(b, e / nc, c0 + e % nc);
            }
            __syncthreads();
            if (tid < DET_PIX) {
                if (nc == DET_CH) {
#pragma unroll
                    for (int cc = 0; cc < DET_CH; cc += 4) {
                        const float4 v = *reinterpret_cast<const float4*>(&slab[tid][cc]);
                        s = s + v.x; s = s + v.y; s = s + v.z; s = s + v.w;
                    }
                } else
                    for (int cc = 0; cc < nc; ++cc) s = s + slab[tid][cc];
            }
            __syncthreads();
        }
    }
    if (tid < DET_PIX && p0 + tid < HW) pixel_put(s, p0 + tid, B * C, d_out, accumulate, threshold, pix);
}

// four consecutive channels as floats
__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4(const bf16_t* p) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    return make_float4(lo16(v.x), hi16(v.x), lo16(v.y), hi16(v.y));
}

template <typename T, int C4>
__global__ __launch_bounds__(64) void pixel_diff_vec_kernel(const T* __restrict__ cached, const T* __restrict__ fresh, int B, int HW,
                                                            float* __restrict__ d_out, int accumulate, float threshold,
                                                            uint8_t* __restrict__ pix) {
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (p >= HW) return;
    float s = 0.f;
#pragma unroll 2
    for (int b = 0; b < B; ++b) {
        const size_t off = ((size_t)b * HW + p) * (4 * C4);
        float4 x[C4], y[C4];
#pragma unroll
        for (int q = 0; q < C4; ++q) { x[q] = load4(cached + off + 4 * q); y[q] = load4(fresh + off + 4 * q); }
#pragma unroll
        for (int q = 0; q < C4; ++q) {
            s = s + fabsf(y[q].x - x[q].x); s = s + fabsf(y[q].y - x[q].y); s = s + fabsf(y[q].z - x[q].z); s = s + fabsf(y[q].w - x[q].w);
        }
    }
    pixel_put(s, p, B * 4 * C4, d_out, accumulate, threshold, pix);
}

template <typename T>
static void launch_pixel_diff(const void* cached, const void* fresh, int B, int HW, int C, float* d_out, int accumulate, float threshold,
                              uint8_t* pix, hipStream_t st) {
    const T* a = (const T*)cached; const T* b = (const T*)fresh;
    // vectors of four channels lie on multiples of their size where the maps do
    const bool vec = C % 4 == 0 && C <= 16 && (reinterpret_cast<uintptr_t>(cached) | reinterpret_cast<uintptr_t>(fresh)) % (4 * sizeof(T)) == 0;
    const dim3 vgrid(ceil_div(HW, 64)), vblock(64);
    if (vec && C == 4) hipLaunchKernelGGL((pixel_diff_vec_kernel<T, 1>), vgrid, vblock, 0, st, a, b, B, HW, d_out, accumulate, threshold, pix);
    else if (vec && C == 8) hipLaunchKernelGGL((pixel_diff_vec_kernel<T, 2>), vgrid, vblock, 0, st, a, b, B, HW, d_out, accumulate, threshold, pix);
    else if (vec && C == 12) hipLaunchKernelGGL((pixel_diff_vec_kernel<T, 3>), vgrid, vblock, 0, st, a, b, B, HW, d_out, accumulate, threshold, pix);
    else if (vec) hipLaunchKernelGGL((pixel_diff_vec_kernel<T, 4>), vgrid, vblock, 0, st, a, b, B, HW, d_out, accumulate, threshold, pix);
    else if (HW <= 64 * 128)
        hipLaunchKernelGGL((pixel_diff_kernel<T, 16>), dim3(ceil_div(HW, 16)), dim3(DET_THREADS), 0, st, a, b, B, HW, C, d_out, accumulate, threshold, pix);
    else
        hipLaunchKernelGGL((pixel_diff_kernel<T, 64>), dim3(ceil_div(HW, 64)), dim3(DET_THREADS), 0, st, a, b, B, HW, C, d_out, accumulate, threshold, pix);
}

// ---------------------------------------------------------------------------
// tile OR + ordered compaction, one workgroup; tiles are taken 256 at a time,
// the running base keeps ids ascending across chunks.
// ---------------------------------------------------------------------------
// Word: what a row of a tile is read in (8, 4 or 1 pixels).  One pixel at a time an 8 x 8 tile is a chain of 64 byte loads (64 x 64
// pixels: 4.5 -> 1.9 us).
template <typename Word>
__global__ __launch_bounds__(256) void tile_compact_kernel(const uint8_t* __restrict__ pix, int H, int W, int tile_h, int tile_w,
                                                           uint8_t* __restrict__ tile_mask, int* __restrict__ idx,
                                                           int capacity, int* __restrict__ n_active) {
    __shared__ int wave_cnt[4];
    const int tw = W / tile_w, nt = tw * (H / tile_h);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int c0 = 0; c0 < nt; c0 += 256) {
        const int t = c0 + threadIdx.x;
        bool act = false;
        if (t < nt) {
            const int y0 = (t / tw) * tile_h, x0 = (t % tw) * tile_w;
            Word any = 0;
            if (tile_h == 8 && tile_w == (int)sizeof(Word)) {           // all rows in flight at once
#pragma unroll
                for (int yy = 0; yy < 8; ++yy) any |= *reinterpret_cast<const Word*>(pix + (y0 + yy) * W + x0);
            } else {
                for (int yy = 0; yy < tile_h; ++yy)
                    for (int xx = 0; xx < tile_w; xx += (int)sizeof(Word)) any |= *reinterpret_cast<const Word*>(pix + (y0 + yy) * W + x0 + xx);
            }
            act = any != 0;
            tile_mask[t] = act ? 1 : 0;
        }
        const unsigned long long bal = __ballot(act);
        const int before = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wave_cnt[wave] = __popcll(bal);
        __syncthreads();
        int off = base, total = 0;
        for (int w = 0; w < 4; ++w) {
            if (w < wave) off += wave_cnt[w];
            total += wave_cnt[w];
        }
        if (act) {
            const int pos = off + before;
            if (pos < capacity) idx[pos] = t;
        }
        base += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *n_active = base;
}

static void launch_tile_compact(const uint8_t* pix, int H, int W, int tile_h, int tile_w, uint8_t* tile_mask, int* idx, int capacity,
                                int* n_active, hipStream_t st) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(pix);              // W is a multiple of tile_w: rows of tiles start on multiples of the word
    if (tile_w % 8 == 0 && at % 8 == 0)
        hipLaunchKernelGGL(tile_compact_kernel<unsigned long long>, dim3(1), dim3(256), 0, st, pix, H, W, tile_h, tile_w, tile_mask, idx, capacity, n_active);
    else if (tile_w % 4 == 0 && at % 4 == 0)
        hipLaunchKernelGGL(tile_compact_kernel<unsigned>, dim3(1), dim3(256), 0, st, pix, H, W, tile_h, tile_w, tile_mask, idx, capacity, n_active);
    else
        hipLaunchKernelGGL(tile_compact_kernel<uint8_t>, dim3(1), dim3(256), 0, st, pix, H, W, tile_h, tile_w, tile_mask, idx, capacity, n_active);
}

__global__ void or_pool_kernel(const uint8_t* __restrict__ m, int H, int W, uint8_t* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int Ho = H / 2, Wo = W / 2;
    if (i >= Ho * Wo) return;
    const int y = i / Wo, x = i % Wo;
    const uint8_t* r0 = m + (2 * y) * W + 2 * x;
    out[i] = (r0[0] | r0[1] | r0[W] | r0[W + 1]) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// Otsu in two launches.  Values are min-max normalised in double; bin k of 257 holds values with floor(256 v) == k, so
// class A of threshold k/256 is exactly bins [0, k).  Every bin's sum is taken in index order: the order is part of the
// result, so the fullest bin (2082 of 4096 values in an edit's mask) is what bounds this: a chain of dependent additions, 16 cycles each, unless
// they are rounded ahead (ordered_sum.h: a round of ~900 cycles for 256 of them instead of 4100).
//  - otsu_bins_kernel: four bins per workgroup of sixteen waves.  The waves normalise 4096 values in registers, pack those of each bin behind one
//    another in LDS (ballots, the waves' counts scanned in between by one lane each), and one wave per bin adds them up from there.
//  - otsu_apply_kernel: every workgroup finds the threshold for itself (the sums below a bin one chain of 257 additions, the counts
//    below it, whole numbers, a scan, the objectives a bin per thread) and thresholds its share of the values.
// us, added one by one and now: bins 18.9 -> 16.0 for 64 x 64 values; with the threshold, five steps of 64 x 64 25.9 -> 21.3, of 96 x 96 48.1 -> 34.1; a whole mask
// of five steps at 64 x 64 takes the host 40 to launch either way.
// ---------------------------------------------------------------------------
constexpr int OTSU_BINS = 257, OTSU_CHUNK = 4096, OTSU_WG_BINS = 4, OTSU_WAVES = 16;
struct OtsuWs { double lo, hi; double cnt[OTSU_BINS]; double sum[OTSU_BINS]; };

#if defined(__HIP_DEVICE_COMPILE__)
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_or_zero(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false), hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
// A wavefront for ordered_sum.
struct Wavefront {
    using Lanes = double;
    static __device__ __forceinline__ int lane() { return __lane_id(); }
    static __device__ __forceinline__ double zero() { return 0.0; }
    static __device__ __forceinline__ double abs(double x) { return fabs(x); }
    static __device__ __forceinline__ unsigned long long ballot(bool c) { return __ballot(c); }
    static __device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
    static __device__ __forceinline__ double at(double x, int lane) {
        const long long b = __double_as_longlong(x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
        return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
    }
    static __device__ __forceinline__ double from(double x, int first) { return lane() < first ? 0.0 : x; }
    static __device__ __forceinline__ double before(double x) { return dpp_or_zero<0x138, 0xf>(x); }
    static __device__ __forceinline__ double scan(double x) {
        x += dpp_or_zero<0x111, 0xf>(x); x += dpp_or_zero<0x112, 0xf>(x); x += dpp_or_zero<0x114, 0xf>(x); x += dpp_or_zero<0x118, 0xf>(x);
        x += dpp_or_zero<0x142, 0xa>(x); x += dpp_or_zero<0x143, 0xc>(x);      // lane 15 of a row to the next row, lane 31 to the upper half
        return x;
    }
    static __device__ __forceinline__ void load(double (&x)[4], const double* src, int i0, int total) {
#pragma unroll
        for (int q = 0; q < 4; ++q) { const int i = i0 + lane() * 4 + q; x[q] = src[min(i, total - 1)]; if (i >= total) x[q] = 0.0; }
    }
};
#endif

__global__ __launch_bounds__(64 * OTSU_WAVES) void otsu_bins_kernel(const float* __restrict__ diff, int n, OtsuWs* __restrict__ ws) {
    constexpr int NT = 64 * OTSU_WAVES, PER = OTSU_CHUNK / NT;
    __shared__ __attribute__((aligned(16))) float red_lo[OTSU_WAVES], red_hi[OTSU_WAVES];
    __shared__ int wave_cnt[OTSU_WG_BINS * OTSU_WAVES];
    static_assert(OTSU_WG_BINS * OTSU_WAVES == 64 && OTSU_WAVES == 16, "a lane per bin and wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char otsu_lds[];
    double (*mine)[OTSU_CHUNK + 64] = reinterpret_cast<double (*)[OTSU_CHUNK + 64]>(otsu_lds);      // [OTSU_WG_BINS], zeros behind a bin's values
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), k0 = blockIdx.x * OTSU_WG_BINS;
    float flo = INFINITY, fhi = -INFINITY;
#pragma unroll 4
    for (int i = t; i < n; i += NT) { const float v = diff[i]; flo = fminf(flo, v); fhi = fmaxf(fhi, v); }
    for (int o = 32; o > 0; o >>= 1) { flo = fminf(flo, __shfl_xor(flo, o)); fhi = fmaxf(fhi, __shfl_xor(fhi, o)); }
    if (lane == 0) { red_lo[wave] = flo; red_hi[wave] = fhi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < OTSU_WAVES; w += 4) {
        const float4 l = *reinterpret_cast<const float4*>(&red_lo[w]), h = *reinterpret_cast<const float4*>(&red_hi[w]);
        flo = fminf(flo, fminf(fminf(l.x, l.y), fminf(l.z, l.w)));
        fhi = fmaxf(fhi, fmaxf(fmaxf(h.x, h.y), fmaxf(h.z, h.w)));
    }
    const double lo = fmin(1e300, (double)flo), hi = fmax(-1e300, (double)fhi);
    const double range = hi - lo;
    // n / range, correctly rounded: the quotient by the rounded reciprocal, corrected with its exact remainder (Markstein's theorem); an
    // infinite range has no such remainder
    const double inv = 1.0 / range;
    const bool finite = range <= 1e300;
    auto normalised = [&](double x) {
        const double q = x * inv;
        return finite ? fma(fma(-q, range, x), inv, q) : x / range;
    };
    const int k = k0 + wave;
    double sum = 0.0;
    int count = 0;
    for (int c0 = 0; c0 < n; c0 += OTSU_CHUNK) {
        // wave w holds values c0 + w * 256 .. in index order: PER rows of 64
        double v[PER]; int bin[PER], place[PER], held[OTSU_WG_BINS] = {};
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = c0 + (wave * PER + j) * 64 + lane;
            v[j] = i < n && range > 0 ? normalised((double)diff[i] - lo) : 0.0;
            bin[j] = i < n ? (int)floor(v[j] * 256.0) - k0 : -1;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {                        // place among this wave's values of the bin
            unsigned long long own = 0;
            place[j] = 0;
#pragma unroll
            for (int b = 0; b < OTSU_WG_BINS; ++b) {
                const unsigned long long bal = __ballot(bin[j] == b);
                if (bin[j] == b) { own = bal; place[j] = held[b]; }
                held[b] += __popcll(bal);
            }
            place[j] += __builtin_amdgcn_mbcnt_hi((unsigned)(own >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)own, 0));
        }
        if (lane < OTSU_WG_BINS) wave_cnt[lane * OTSU_WAVES + wave] = lane == 0 ? held[0] : lane == 1 ? held[1] : lane == 2 ? held[2] : held[3];
        __syncthreads();
        // lane 16 b + w: values of bin b in the waves up to w
        const int c = wave_cnt[lane];
        int upto = c;
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false); upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false); upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);
        int base[OTSU_WG_BINS], total = 0;                     // total: of bin `wave` in the first waves
#pragma unroll
        for (int b = 0; b < OTSU_WG_BINS; ++b) {
            base[b] = __builtin_amdgcn_readlane(upto - c, b * OTSU_WAVES + wave);
            const int all = __builtin_amdgcn_readlane(upto, b * OTSU_WAVES + OTSU_WAVES - 1);
            if (wave == b) total = all;
            if (wave == OTSU_WG_BINS + b) mine[b][all + lane] = 0.0;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if ((unsigned)bin[j] < (unsigned)OTSU_WG_BINS) mine[bin[j]][(bin[j] == 0 ? base[0] : bin[j] == 1 ? base[1] : bin[j] == 2 ? base[2] : base[3]) + place[j]] = v[j];
        __syncthreads();
        if (wave < OTSU_WG_BINS) {
#if defined(__HIP_DEVICE_COMPILE__)
            sum = ordered_sum<Wavefront>(sum, static_cast<const double*>(mine[wave]), total, k < OTSU_BINS - 1 ? (k + 1) / 256.0 : 1.0);
#endif
            count += total;
        }
        __syncthreads();
    }
    if (lane == 0 && wave < OTSU_WG_BINS && k < OTSU_BINS) { ws->cnt[k] = (double)count; ws->sum[k] = sum; }
    if (blockIdx.x == 0 && t == 0) { ws->lo = lo; ws->hi = hi; }
}

__global__ __launch_bounds__(256) void otsu_apply_kernel(const float* __restrict__ diff, int n, float* __restrict__ eps_out,
                                                         uint8_t* __restrict__ pix, const OtsuWs* __restrict__ ws) {
    __shared__ double sum[OTSU_BINS + 15], cnt_lo[OTSU_BINS], sum_lo[OTSU_BINS], total[2], wave_best[4];      // _lo: sums over the bins below k
    const int t = threadIdx.x, lane = t & 63;
    __shared__ int wave_k[4];
    const double lo = ws->lo, range = ws->hi - lo;
    for (int k = t; k < OTSU_BINS; k += 256) sum[k] = ws->sum[k];
    double c4[4];                                              // second wave: counts of bins 4 lane .. 4 lane + 3
    if (t >> 6 == 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) c4[q] = ws->cnt[4 * lane + q];
    __syncthreads();
    if (t >> 6 == 1) {                                         // counts are whole numbers: any order gives their sum
        double up = c4[0] + c4[1] + c4[2] + c4[3], mine = up;
        for (int o = 1; o < 64; o <<= 1) { const double x = __shfl_up(up, o); if (lane >= o) up += x; }
        double below = up - mine;
#pragma unroll
        for (int q = 0; q < 4; ++q) { cnt_lo[4 * lane + q] = below; below += c4[q]; }
        if (lane == 63) { cnt_lo[OTSU_BINS - 1] = below; total[0] = below + ws->cnt[OTSU_BINS - 1]; }
    }
    if (t == 0) {
        double s = 0, sk[16], next[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) sk[q] = sum[q];
        for (int k0 = 0; k0 < OTSU_BINS - 1; k0 += 16) {       // sixteen bins' reads ahead of the additions
#pragma unroll
            for (int q = 0; q < 16; ++q) next[q] = sum[k0 + 16 + q];        // (past the last bin: not used)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 16; ++q) { sum_lo[k0 + q] = s; s += sk[q]; }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 16; ++q) sk[q] = next[q];
        }
        sum_lo[OTSU_BINS - 1] = s;
        total[1] = s + sum[OTSU_BINS - 1];
    }
    __syncthreads();
    // the first bin with the largest objective: a bin per thread, the last one as the last wave's second
    double best = -1.0;
    int best_k = 0;
    for (int k = t; k < OTSU_BINS; k += t == 255 ? 1 : OTSU_BINS) {
        const double ca = cnt_lo[k], sa = sum_lo[k], cb = total[0] - ca, sb = total[1] - sa;
        double o = 0.0;
        if (ca > 0 && cb > 0) {
            const double dm = sa / ca - sb / cb;
            o = ca * cb / (total[0] * total[0]) * dm * dm;
        }
        if (o > best) { best = o; best_k = k; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double b2 = __shfl_xor(best, o);
        const int k2 = __shfl_xor(best_k, o);
        if (b2 > best || (b2 == best && k2 < best_k)) { best = b2; best_k = k2; }
    }
    if (lane == 0) { wave_best[t >> 6] = best; wave_k[t >> 6] = best_k; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w)
        if (wave_best[w] > best || (wave_best[w] == best && wave_k[w] < best_k)) { best = wave_best[w]; best_k = wave_k[w]; }
    if (t == 0 && blockIdx.x == 0) *eps_out = (float)(best_k / 256.0);
    const double eps = best_k / 256.0;
    for (int i = blockIdx.x * 256 + t; i < n; i += gridDim.x * 256) {
        const double v = range > 0 ? ((double)diff[i] - lo) / range : 0.0;
        pix[i] = v >= eps ? 1 : 0;
    }
}

// one workgroup per candidate block size (h, w) = (2<<i, 2<<j)
__global__ __launch_bounds__(256) void apsc_count_kernel(const uint8_t* __restrict__ pix, int H, int W,
                                                         int* __restrict__ counts) {
    __shared__ int red[256];
    const int h = 2 << (blockIdx.x / 5), w = 2 << (blockIdx.x % 5);
    if (H % h || W % w) { if (threadIdx.x == 0) counts[blockIdx.x] = -1; return; }
    const int bw = W / w, nb = bw * (H / h);
    int c = 0;
    for (int bidx = threadIdx.x; bidx < nb; bidx += 256) {
        const int y0 = (bidx / bw) * h, x0 = (bidx % bw) * w;
        bool any = false;
        for (int yy = 0; yy < h && !any; ++yy)
            for (int xx = 0; xx < w; ++xx) if (pix[(y0 + yy) * W + x0 + xx]) { any = true; break; }
        c += any;
    }
    red[threadIdx.x] = c;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) { if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s]; __syncthreads(); }
    if (threadIdx.x == 0) counts[blockIdx.x] = red[0];
}

static int check_map(const char* fn, const void* a, const void* b, int dtype, int B, int H, int W, int C) {
    if (!a || !b) return fail(FISE_ERR_NULL, "%s: null map pointer", fn);
    if (dtype != FISE_F32 && dtype != FISE_BF16) return fail(FISE_ERR_DTYPE, "%s: dtype %d", fn, dtype);
    if (B < 1 || H < 1 || W < 1 || C < 1) return fail(FISE_ERR_SHAPE, "%s: bad shape B%d H%d W%d C%d", fn, B, H, W, C);
    return FISE_OK;
}
static int check_tile(const char* fn, int H, int W, int tile) {
    if (tile < 1 || H < 1 || W < 1 || H % tile || W % tile)
        return fail(FISE_ERR_SHAPE, "%s: H=%d, W=%d must be positive multiples of tile=%d", fn, H, W, tile);
    return FISE_OK;
}

}  // namespace fise

using namespace fise;

extern "C" int fise_mask_from_pixels(const uint8_t* pix_mask, int H, int W, int tile, uint8_t* tile_mask,
                                     int32_t* tile_idx, int capacity, int32_t* n_active, void* stream) {
    if (!pix_mask || !tile_mask || !tile_idx || !n_active) return fail(FISE_ERR_NULL, "fise_mask_from_pixels: null pointer");
    if (int e = check_tile("fise_mask_from_pixels", H, W, tile)) return e;
    if (capacity < 0) return fail(FISE_ERR_CAPACITY, "fise_mask_from_pixels: capacity %d", capacity);
    launch_tile_compact(pix_mask, H, W, tile, tile, tile_mask, tile_idx, capacity, n_active, as_stream(stream));
    FISE_CHECK_LAUNCH("fise_mask_from_pixels");
    return FISE_OK;
}

extern "C" int fise_mask_from_pixels_rect(const uint8_t* pix_mask, int H, int W, int tile_h, int tile_w, uint8_t* tile_mask,
                                          int32_t* tile_idx, int capacity, int32_t* n_active, void* stream) {
    if (!pix_mask || !tile_mask || !tile_idx || !n_active) return fail(FISE_ERR_NULL, "fise_mask_from_pixels_rect: null pointer");
    if (tile_h < 1 || tile_w < 1 || H < 1 || W < 1 || H % tile_h || W % tile_w)
        return fail(FISE_ERR_SHAPE, "fise_mask_from_pixels_rect: H=%d, W=%d must be positive multiples of the %dx%d block", H, W,
                    tile_h, tile_w);
    if (capacity < 0) return fail(FISE_ERR_CAPACITY, "fise_mask_from_pixels_rect: capacity %d", capacity);
    launch_tile_compact(pix_mask, H, W, tile_h, tile_w, tile_mask, tile_idx, capacity, n_active, as_stream(stream));
    FISE_CHECK_LAUNCH("fise_mask_from_pixels_rect");
    return FISE_OK;
}

extern "C" int fise_mask_detect(const void* cached, const void* fresh, int dtype, int B, int H, int W, int C,
                                float threshold, int tile, uint8_t* pix_mask, uint8_t* tile_mask, int32_t* tile_idx,
                                int capacity, int32_t* n_active, void* stream) {
    if (int e = check_map("fise_mask_detect", cached, fresh, dtype, B, H, W, C)) return e;
    if (!pix_mask || !tile_mask || !tile_idx || !n_active) return fail(FISE_ERR_NULL, "fise_mask_detect: null output pointer");
    if (int e = check_tile("fise_mask_detect", H, W, tile)) return e;
    if (capacity < 0) return fail(FISE_ERR_CAPACITY, "fise_mask_detect: capacity %d", capacity);
    const int HW = H * W;
    if (dtype == FISE_F32) launch_pixel_diff<float>(cached, fresh, B, HW, C, nullptr, 0, threshold, pix_mask, as_stream(stream));
    else launch_pixel_diff<bf16_t>(cached, fresh, B, HW, C, nullptr, 0, threshold, pix_mask, as_stream(stream));
    FISE_CHECK_LAUNCH("fise_mask_detect(diff)");
    return fise_mask_from_pixels(pix_mask, H, W, tile, tile_mask, tile_idx, capacity, n_active, stream);
}

extern "C" int fise_diff_accumulate(const void* cached, const void* fresh, int dtype, int B, int H, int W, int C,
                                    float* diff_acc, void* stream) {
    if (int e = check_map("fise_diff_accumulate", cached, fresh, dtype, B, H, W, C)) return e;
    if (!diff_acc) return fail(FISE_ERR_NULL, "fise_diff_accumulate: null diff_acc");
    const int HW = H * W;
    if (dtype == FISE_F32) launch_pixel_diff<float>(cached, fresh, B, HW, C, diff_acc, 1, 0.f, nullptr, as_stream(stream));
    else launch_pixel_diff<bf16_t>(cached, fresh, B, HW, C, diff_acc, 1, 0.f, nullptr, as_stream(stream));
    FISE_CHECK_LAUNCH("fise_diff_accumulate");
    return FISE_OK;
}

extern "C" int fise_mask_downsample(const uint8_t* mask, int H, int W, uint8_t* out, void* stream) {
    if (!mask || !out) return fail(FISE_ERR_NULL, "fise_mask_downsample: null pointer");
    if (H < 2 || W < 2 || (H & 1) || (W & 1)) return fail(FISE_ERR_SHAPE, "fise_mask_downsample: H=%d W=%d must be even", H, W);
    const int n = (H / 2) * (W / 2);
    hipLaunchKernelGGL(or_pool_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, as_stream(stream), mask, H, W, out);
    FISE_CHECK_LAUNCH("fise_mask_downsample");
    return FISE_OK;
}

extern "C" size_t fise_otsu_workspace_bytes(void) { return align256(sizeof(OtsuWs)); }

extern "C" int fise_otsu_mask(const float* diff, int n, float* eps_out, uint8_t* pix_mask, void* workspace, void* stream) {
    if (!diff || !eps_out || !pix_mask || !workspace) return fail(FISE_ERR_NULL, "fise_otsu_mask: null pointer");
    if (n < 1) return fail(FISE_ERR_SHAPE, "fise_otsu_mask: n=%d", n);
    constexpr int lds = OTSU_WG_BINS * (OTSU_CHUNK + 64) * (int)sizeof(double);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&otsu_bins_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "fise_otsu_mask: cannot raise the dynamic LDS limit");
    hipLaunchKernelGGL(otsu_bins_kernel, dim3(ceil_div(OTSU_BINS, OTSU_WG_BINS)), dim3(64 * OTSU_WAVES), lds, as_stream(stream), diff, n, (OtsuWs*)workspace);
    FISE_CHECK_LAUNCH("fise_otsu_mask(bins)");
    hipLaunchKernelGGL(otsu_apply_kernel, dim3(std::min(ceil_div(n, 256), 64)), dim3(256), 0, as_stream(stream), diff, n, eps_out, pix_mask,
                       (const OtsuWs*)workspace);
    FISE_CHECK_LAUNCH("fise_otsu_mask");
    return FISE_OK;
}

extern "C" int fise_apsc_block_counts(const uint8_t* pix_mask, int H, int W, int32_t* counts, void* stream) {
    if (!pix_mask || !counts) return fail(FISE_ERR_NULL, "fise_apsc_block_counts: null pointer");
    if (H < 1 || W < 1) return fail(FISE_ERR_SHAPE, "fise_apsc_block_counts: H=%d W=%d", H, W);
    hipLaunchKernelGGL(apsc_count_kernel, dim3(25), dim3(256), 0, as_stream(stream), pix_mask, H, W, counts);
    FISE_CHECK_LAUNCH("fise_apsc_block_counts");
    return FISE_OK;
}

extern "C" int fise_apsc_select(const int32_t* counts, int kh, int kw, int* h, int* w, int64_t* cost) {
    if (!counts || !h || !w) return fail(FISE_ERR_NULL, "fise_apsc_select: null pointer");
    if (kh < 1 || kw < 1) return fail(FISE_ERR_SHAPE, "fise_apsc_select: kernel %dx%d", kh, kw);
    int64_t best = -1;
    for (int i = 0; i < 5; ++i)
        for (int j = 0; j < 5; ++j) {
            const int32_t n = counts[i * 5 + j];
            if (n < 0) continue;
            const int bh = 2 << i, bw = 2 << j;
            const int64_t c = (int64_t)(bh + kh - 1) * (bw + kw - 1) * n;
            if (best < 0 || c < best) { best = c; *h = bh; *w = bw; }
        }
    if (best < 0) return fail(FISE_ERR_SHAPE, "fise_apsc_select: no candidate block size divides the map");
    if (cost) *cost = best;
    return FISE_OK;
}
