// Cross-attention sub-layer of 320 channels and eight heads over the few keys of a prompt, as one launch:
//
//   y = x + Wo attention(Wq LN(x), K, V) + bo
//
// Everything behind the LayerNorm belongs to one row, so a workgroup takes 32 rows of a batch element from the normalisation to the sum, and nothing of
// it goes through memory.  Eight waves, a head each:
//  - The rows are normalised into LDS as bf16, every wave four of them.
//  - A wave multiplies its head's 40 rows of Wq with them, then 40 rows of Wo with the heads' outputs: ten stages of 64 channels through a ring of
//    its own (LDS-direct loads of eight rows of 128 bytes), so that the rows of Wo travel under the attention.  No barrier in between.
//  - Queries, probabilities and outputs never leave the wave's registers: 16 x 16 x 32 products whose rows are numbered so that a result is the next
//    product's operand (row r of a pair of tiles is channel, or key, 8 (r / 4) + r % 4, and that + 4).  Keys, values and the residual are requested up
//    front.
//  - The heads' outputs meet in the place of the normalised rows (the two barriers beside the one behind the normalisation).
// Bound by the 500 KB a workgroup brings in (410 of weights at the ~60 GB/s that loads of eight rows get a CU, keys, values and residual in pieces of 64
// bytes); first touches of the later stages' lines are worth 1.3 us with cold weights.  Against the three launches it stands for (normalisation and
// queries, attention over 77 keys, product and sum), us with warm weights: 1536 rows of a map 17.3 -> 12.6, 5504 29.3 -> 13.6, 8192 32.8 -> 14.4; steps of 12 of 64
// tiles 2247 -> 2214, 43 of 144 4152 -> 4112, dense pass 4950 -> 4878.
#include <cmath>
#include <type_traits>
#include "attention_choice.h"
#include "igemm.h"
#include "profile.h"

namespace fise {

struct CrossDev {
    CrossArgs a;
    int gx; float scale_log2e;
    FastDiv d_gx, d_tiles, d_tt, d_tile, d_tiles_w;
};

#if defined(__HIP_DEVICE_COMPILE__)
// over the four lanes l16, l16 + 16, + 32, + 48
__device__ __forceinline__ float quad_max(float x) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float quad_sum(float x) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
__device__ __forceinline__ bf16x8_t pack8(const f32x4_t& x, const f32x4_t& y) { return __builtin_bit_cast(bf16x8_t, u32x4_t{f2bf2(x[0], x[1]), f2bf2(x[2], x[3]), f2bf2(y[0], y[1]), f2bf2(y[2], y[3])}); }

// Softmax of a lane's row, whose raw scores over keys 32 p + 8 lq + 0 .. 7 and 64 + 4 lq + 0 .. 3 are s: probabilities against the largest of their 32 keys as operands, and
// what the product of each operand with the values counts for.  One weight in 32 is then exactly one, as where a wave of attention_few_kernel has those keys;
// against the largest of all keys one in 77 is, and the error against 64 bits of a layer of 128 rows x 320 channels 1.743e-3 for 1.738e-3.  (What the rounding leaves of a probability as a
// second operand made it 1.724e-3 for the same time, but an infinite value times a zero there is no number.)
struct KeyWeights { bf16x8_t p[3]; float w[3]; };
__device__ __forceinline__ KeyWeights key_weights(f32x4_t (&s)[CROSS_KEYS / 16], int n_ctx, int lq, float scale_log2e) {
    KeyWeights r;
    float top[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        top[p] = -INFINITY;
#pragma unroll
        for (int t = 2 * p; t < 2 * p + 2 && t < CROSS_KEYS / 16; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = p < 2 ? 32 * p + 8 * lq + 4 * (t & 1) + e : 64 + 4 * lq + e;
                s[t][e] = key < n_ctx ? s[t][e] : -INFINITY;
                top[p] = fmaxf(top[p], s[t][e]);
            }
        top[p] = quad_max(top[p]);
    }
    const float mx = fmaxf(fmaxf(top[0], top[1]), top[2]);
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const float m = (top[p] > -INFINITY ? top[p] : mx) * scale_log2e;       // no such keys: probabilities of zero
        float part = 0.f;
#pragma unroll
        for (int t = 2 * p; t < 2 * p + 2 && t < CROSS_KEYS / 16; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) { s[t][e] = __builtin_amdgcn_exp2f(fmaf(s[t][e], scale_log2e, -m)); part += s[t][e]; }
        r.w[p] = __builtin_amdgcn_exp2f(m - mx * scale_log2e);
        sum += part * r.w[p];
        r.p[p] = pack8(s[2 * p], p < 2 ? s[2 * p + 1] : f32x4_t{0.f, 0.f, 0.f, 0.f});
    }
    const float inv = 1.0f / quad_sum(sum);
#pragma unroll
    for (int p = 0; p < 3; ++p) r.w[p] *= inv;
    return r;
}
// Sixteen channels of the values (of keys 32 p ..), weighted.
__device__ __forceinline__ f32x4_t weighted(const u32x4_t& v0, const u32x4_t& v1, const u32x4_t& v2, const KeyWeights& k) {
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v0), k.p[0], zero, 0, 0, 0) * k.w[0] +
           __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v1), k.p[1], zero, 0, 0, 0) * k.w[1] +
           __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, v2), k.p[2], zero, 0, 0, 0) * k.w[2];
}
#endif

// MAP: rows are pixels of bf16 maps (in and out), else compact float rows, updated in place.
template <bool MAP>
__global__ __launch_bounds__(512, 2) void cross_attention_kernel(const CrossDev g) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int C = CROSS_C, D = C / CROSS_HEADS, BM = 32, PITCH = 2 * C, ND = 3, PIECES = D / 8, STAGE = D * 128, NT = CROSS_KEYS / 16, TOUCH = 2;
    constexpr unsigned OOB = 0x80000000u;
    static_assert(D == 40 && NT == 5, "numbering of rows and keys");
    const CrossArgs& a = g.a;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    unsigned char* const ring = lds + BM * PITCH;
    int* const rowpix = reinterpret_cast<int*>(ring + CROSS_HEADS * ND * STAGE);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // every XCD gets a contiguous run of row tiles
    const int chunk = (int)gridDim.x >> 3;
    int w = blockIdx.x;
    if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
    const int b = (int)fdiv((unsigned)w, g.d_gx), m0 = (w - b * g.gx) * BM;

    // ---- rows: sixteen lanes a row, five pieces of four channels each
    const int row = wave * 4 + lq;
    const unsigned i_row = (unsigned)min(m0 + row, a.Ma - 1);
    f32x4_t v[5];
    if constexpr (MAP) {
        const unsigned t = fdiv(i_row, g.d_tt), rp = i_row - t * (unsigned)(a.tile * a.tile), id = (unsigned)((const FISE_AS1 int*)a.tile_idx)[t];
        const unsigned py = fdiv(rp, g.d_tile), ty = fdiv(id, g.d_tiles_w);
        const unsigned pix = (ty * a.tile + py) * (unsigned)a.W + (id - ty * a.tiles_w) * a.tile + (rp - py * a.tile);
        if (l16 == 0) rowpix[row] = (int)pix;
        const FISE_AS1 u32x2_t* q = (const FISE_AS1 u32x2_t*)((const bf16_t*)a.x + ((size_t)b * a.HW + pix) * C) + l16;
#pragma unroll
        for (int j = 0; j < 5; ++j) { const u32x2_t u = q[j * 16]; v[j] = f32x4_t{__uint_as_float(u.x), __uint_as_float(u.y), 0.f, 0.f}; }
    } else {
        const FISE_AS1 f32x4_t* q = (const FISE_AS1 f32x4_t*)((const float*)a.x + ((size_t)b * a.Ma + i_row) * C) + l16;
#pragma unroll
        for (int j = 0; j < 5; ++j) v[j] = q[j * 16];
    }
    u32x2_t gam[5], bet[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        gam[j] = ((const FISE_AS1 u32x2_t*)a.gamma)[j * 16 + l16];
        bet[j] = ((const FISE_AS1 u32x2_t*)a.beta)[j * 16 + l16];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- weights: stages 0 - 4 are this head's rows of Wq, 5 - 9 as many of Wo.  Slot p of row r holds segment p ^ ((r >> 1) & 7).
    const unsigned seg = (unsigned)((lane & 7) ^ (lane >> 4)) * 16u, vd = (unsigned)(lane >> 3) * PITCH;
    unsigned char* const my_ring = ring + wave * (ND * STAGE);
    auto load = [&](int s) {
        const __amdgpu_buffer_rsrc_t rs = buf(s < 5 ? a.wq : a.wo, C * PITCH);
#pragma unroll
        for (int p = 0; p < PIECES; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (FISE_AS3 void*)(my_ring + (s % ND) * STAGE + p * 1024), 16, vd + (p & 1 ? seg ^ 64u : seg),
                                                     (unsigned)((wave * D + p * 8) * PITCH + (s % 5) * 128), 0, 0);
    };
    // Later stages' lines are cold for all workgroups of an XCD at once: they touch them first, each a share (one dword a line, into the ring before it is filled).
    {
        constexpr int LINES = C * 2 + C * 5;               // stages 3 and 4 of Wq, then Wo
        const int per_xcd = max(1, chunk), me = chunk ? w % chunk : 0;
#pragma unroll
        for (int k = 0; k < TOUCH; ++k) {
            const int q = ((k * per_xcd + me) * CROSS_HEADS + wave) * 64 + lane;
            const bool o = q >= C * 2;
            const int r = o ? q - C * 2 : q;
            const unsigned at = o ? (unsigned)r * 128u : (unsigned)((r >> 1) * PITCH + (3 + (r & 1)) * 128);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buf(a.wq, C * PITCH), (FISE_AS3 void*)my_ring, 4, o ? OOB : at, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buf(a.wo, C * PITCH), (FISE_AS3 void*)my_ring, 4, o && q < LINES ? at : OOB, 0, 0, 0);
        }
    }
#pragma unroll
    for (int s = 0; s < ND; ++s) load(s);
    __builtin_amdgcn_sched_barrier(0);

    // ---- LayerNorm
    {
        f32x4_t x[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            x[j] = v[j];
            if constexpr (MAP) {
                const unsigned w0 = __float_as_uint(v[j].x), w1 = __float_as_uint(v[j].y);
                x[j] = f32x4_t{lo16(w0), hi16(w0), lo16(w1), hi16(w1)};
            }
        }
        layer_norm<16>(x, gam, bet, a.eps);
        put_row<16>(lds + row * PITCH, row, l16, x);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // not the loads in flight

    // ---- keys (row r of tile 2p + h is key 32 p + 8 (r / 4) + 4 h + r % 4; of the last tile 64 + r) and values: keys that do not exist are zeros
    u32x4_t k16[NT], v16[3][2]; u32x2_t k8[NT], v8[3];
    auto fetch_keys = [&]() {
        const __amdgpu_buffer_rsrc_t rk = buf(a.K + (size_t)b * a.n_ctx * C, (unsigned)(a.n_ctx * PITCH)), rv = buf(a.Vt + (size_t)b * C * a.n_stride, (unsigned)(C * a.n_stride) * 2u);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int key = t < NT - 1 ? 32 * (t >> 1) + 8 * (l16 >> 2) + 4 * (t & 1) + (l16 & 3) : 64 + l16;
            const unsigned off = key < a.n_ctx ? (unsigned)(key * PITCH + wave * (2 * D)) : OOB;
            k16[t] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rk, off + lq * 16u, 0, 0));
            k8[t] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rk, lq < 2 ? off + 64u + lq * 8u : OOB, 0, 0));
        }
#pragma unroll
        for (int dt = 0; dt < 3; ++dt) {
            const int d = dt * 16 + l16;
            const unsigned off = (unsigned)((wave * D + d) * a.n_stride) * 2u;
#pragma unroll
            for (int p = 0; p < 2; ++p) v16[dt][p] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rv, d < D && 32 * p + 8 * lq < a.n_ctx ? off + (unsigned)(64 * p + 16 * lq) : OOB, 0, 0));
            v8[dt] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rv, d < D && 64 + 4 * lq < a.n_ctx ? off + (unsigned)(128 + 8 * lq) : OOB, 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
    };


    // ---- product of 48 rows of a head's weights (the last eight twice) and the 32 rows in LDS over five stages
    const unsigned rx = (unsigned)(l16 * PITCH + ((lq ^ ((l16 >> 1) & 7)) * 16));
    auto product = [&](auto first, f32x4_t (&acc)[3][2], const int (&wrow)[3], auto behind_first) {
        constexpr int S0 = decltype(first)::value;
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[u][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            constexpr int AFTER = (ND - 1) * PIECES, KV = 2 * NT + 9, EPI = 9;
            const int s = S0 + k;
            // younger loads: two stages; behind those of stage 3 came the keys and values, behind those of stage 7 bias and residual
            if (s == 0 || s == 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AFTER) : "memory");
            else if (s < 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AFTER + KV) : "memory");
            else if (s < 8) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AFTER + EPI) : "memory");
            else if (s == 8) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PIECES) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const unsigned char* const stage = my_ring + (s % ND) * STAGE;
            bf16x8_t fw[2][3], fx[2][2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int u = 0; u < 3; ++u) fw[ks][u] = *reinterpret_cast<const bf16x8_t*>(stage + wrow[u] * 128 + (((lq + 4 * ks) ^ ((wrow[u] >> 1) & 7)) * 16));
#pragma unroll
                for (int i = 0; i < 2; ++i) fx[ks][i] = *reinterpret_cast<const bf16x8_t*>(lds + (rx ^ (ks ? 64u : 0u)) + i * 16 * PITCH + k * 128);
            }
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (s + ND < 10) load(s + ND);
            if (k == 0) behind_first();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int u = 0; u < 3; ++u)
#pragma unroll
                    for (int i = 0; i < 2; ++i) acc[u][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks][u], fx[ks][i], acc[u][i], 0, 0, 0);
        }
    };
    // Four of a lane's eight elements, the rest zeros.  (Not 16 x 16 x 16 products: where a 16 x 16 x 32 product goes on with their sums the compiler leaves
    // too few wait states, and the last two elements of a lane were those of the registers' former contents.)
    auto pack4 = [](const f32x4_t& x) { return __builtin_bit_cast(bf16x8_t, u32x4_t{f2bf2(x[0], x[1]), f2bf2(x[2], x[3]), 0, 0}); };
    auto half = [](const u32x2_t& x) { return __builtin_bit_cast(bf16x8_t, u32x4_t{x.x, x.y, 0, 0}); };
    f32x4_t acc[3][2];
    {
        const int wrow[3] = {8 * (l16 >> 2) + (l16 & 3), 8 * (l16 >> 2) + 4 + (l16 & 3), 32 + (l16 & 7)};
        product(std::integral_constant<int, 0>(), acc, wrow, fetch_keys);
    }

    // ---- attention of this head: lane = row l16 of both row tiles, keys 32 p + 8 lq + 0 .. 7 and 64 + 4 lq + 0 .. 3
    f32x4_t o[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bf16x8_t q32 = pack8(acc[0][i], acc[1][i]);
        const bf16x8_t q8 = pack4(acc[2][i]);               // channels 32 + 4 lq ..; from 40 on the keys hold zeros
        f32x4_t s[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(half(k8[t]), q8, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, k16[t]), q32, s[t], 0, 0, 0);
        }
        const KeyWeights kw = key_weights(s, a.n_ctx, lq, g.scale_log2e);
        auto live = [&](unsigned w, int key) { return key + 1 < a.n_ctx ? w : key < a.n_ctx ? w & 0xffffu : 0u; };       // a word of two keys
#pragma unroll
        for (int dt = 0; dt < 3; ++dt) {
            if (i == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) { v16[dt][0][e] = live(v16[dt][0][e], 8 * lq + 2 * e); v16[dt][1][e] = live(v16[dt][1][e], 32 + 8 * lq + 2 * e); }
                v8[dt].x = live(v8[dt].x, 64 + 4 * lq); v8[dt].y = live(v8[dt].y, 66 + 4 * lq);
            }
            o[dt][i] = weighted(v16[dt][0], v16[dt][1], u32x4_t{v8[dt].x, v8[dt].y, 0, 0}, kw);
        }
    }
    // what the epilogue adds, under the hand-over and the second product
    const int pix[2] = {MAP ? rowpix[l16] : m0 + l16, MAP ? rowpix[16 + l16] : m0 + 16 + l16};
    u32x2_t bias[3]; f32x4_t res[3][2];
    {
        const __amdgpu_buffer_rsrc_t rb = buf(a.bias, a.bias ? 2u * C : 0u);
        const __amdgpu_buffer_rsrc_t rr = MAP ? buf((const bf16_t*)a.x + (size_t)b * a.HW * C, (unsigned)(a.HW * C) * 2u) : buf((const float*)a.x + (size_t)b * a.Ma * C, (unsigned)(a.Ma * C) * 4u);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int col = wave * D + u * 16 + lq * 4;
            bias[u] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rb, (unsigned)col * 2u, 0, 0));
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned no = m0 + i * 16 + l16 < a.Ma && (u < 2 || lq < 2) ? 0u : OOB, at = (unsigned)(pix[i] * C + col);
                if constexpr (MAP) {
                    const u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rr, (at * 2u) | no, 0, 0));
                    res[u][i] = f32x4_t{__uint_as_float(r.x), __uint_as_float(r.y), 0.f, 0.f};
                } else {
                    res[u][i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rr, (at * 4u) | no, 0, 0));
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // the normalised rows have been read
#pragma unroll
    for (int dt = 0; dt < 3; ++dt)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int col = wave * D + dt * 16 + lq * 4, r = i * 16 + l16, sg = col >> 3;
            if (dt < 2 || lq < 2)
                *reinterpret_cast<u32x2_t*>(lds + r * PITCH + (sg >> 3) * 128 + ((sg & 7) ^ ((r >> 1) & 7)) * 16 + (col & 4) * 2) =
                    u32x2_t{f2bf2(o[dt][i][0], o[dt][i][1]), f2bf2(o[dt][i][2], o[dt][i][3])};
        }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x4_t y[3][2];
    {
        const int wrow[3] = {l16, 16 + l16, 32 + (l16 & 7)};
        product(std::integral_constant<int, 5>(), y, wrow, []() {});
    }

#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int col = wave * D + u * 16 + lq * 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = m0 + i * 16 + l16;
            if (m >= a.Ma || (u == 2 && lq >= 2)) continue;
            if constexpr (MAP) {
                const unsigned w0 = __float_as_uint(res[u][i].x), w1 = __float_as_uint(res[u][i].y);
                res[u][i] = f32x4_t{lo16(w0), hi16(w0), lo16(w1), hi16(w1)};
            }
            const f32x4_t z = y[u][i] + f32x4_t{lo16(bias[u].x), hi16(bias[u].x), lo16(bias[u].y), hi16(bias[u].y)} + res[u][i];
            if constexpr (MAP) *(FISE_AS1 u32x2_t*)((bf16_t*)a.out + ((size_t)b * a.HW + pix[i]) * C + col) = u32x2_t{f2bf2(z[0], z[1]), f2bf2(z[2], z[3])};
            else *(FISE_AS1 f32x4_t*)((float*)a.out + ((size_t)b * a.Ma + m) * C + col) = z;
        }
    }
#endif
}

// The same up to the product with Wo, out = attention(Wq LN(x), K, V) as compact bf16 rows, a workgroup per head and 32 rows: 640 channels, whose weights
// are too many for one workgroup, and few rows of 320.  A wave per 64 channels:
//  - it brings that stage of the head's weights into LDS (all of them in flight together, under the normalisation) and multiplies it with the
//    rows; the waves' sums meet in the place of the weights, in wave order, and become queries;
//  - the last two waves hold keys and values and finish sixteen rows each, numbered as above.
// Bound by its start, the rows and 100 KB of weights.  Against a launch each for the queries and the attention, us: transformer block of 160 rows x 640 65.9
// -> 63.1, of 512 82.7 -> 78.5; cross-attention layer of 96 rows x 320 13.0 -> 9.2, of 160 x 640 16.7 -> 12.7; step of 2 of 70 tiles 1787 -> 1755, 12 of 64 2217 -> 2198.
template <int C> struct QueryTile {
    static constexpr int NW = C / 64, D = C / CROSS_HEADS, U = (D + 15) / 16, BM = 32, PITCH = 2 * C + (C % 128 ? 0 : 128), REGION = D * 128 > U * 2048 ? D * 128 : U * 2048,
                         QC = (D + 31) / 32, QPITCH = QC * 64 + 16, LDS = BM * PITCH + NW * REGION;      // QC: 32-wide steps over the head dim
    static_assert(BM * QPITCH <= BM * PITCH, "queries lie in the place of the rows");
};

template <int C, bool MAP>
__global__ __launch_bounds__(C, 1) void query_attention_kernel(const CrossDev g) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = QueryTile<C>;
    constexpr int NW = T::NW, D = T::D, U = T::U, BM = T::BM, PITCH = T::PITCH, NT = CROSS_KEYS / 16, QUADS = BM / 4, PASSES = (QUADS + NW - 1) / NW;
    constexpr unsigned OOB = 0x80000000u;
    const CrossArgs& a = g.a;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    unsigned char* const regions = lds + BM * PITCH;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char* const mine = regions + wave * T::REGION;
    // every XCD gets a contiguous run of (head, row tile), row tiles fastest: the weights of a head are pulled into one L2
    const int chunk = (int)gridDim.x >> 3;
    int w = blockIdx.x;
    if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
    const int tiles = g.gx * a.B, h = (int)fdiv((unsigned)w, g.d_tiles), rt = w - h * tiles, b = (int)fdiv((unsigned)rt, g.d_gx), m0 = (rt - b * g.gx) * BM;

    // ---- rows: sixteen lanes a row, NW pieces of four channels each
    f32x4_t v[PASSES][NW];
    u32x2_t gam[NW], bet[NW];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int quad = p * NW + wave;
        if (quad >= QUADS) continue;
        const unsigned i_row = (unsigned)min(m0 + quad * 4 + lq, a.Ma - 1);
        if constexpr (MAP) {
            const unsigned t = fdiv(i_row, g.d_tt), rp = i_row - t * (unsigned)(a.tile * a.tile), id = (unsigned)((const FISE_AS1 int*)a.tile_idx)[t];
            const unsigned py = fdiv(rp, g.d_tile), ty = fdiv(id, g.d_tiles_w);
            const unsigned pix = (ty * a.tile + py) * (unsigned)a.W + (id - ty * a.tiles_w) * a.tile + (rp - py * a.tile);
            const FISE_AS1 u32x2_t* q = (const FISE_AS1 u32x2_t*)((const bf16_t*)a.x + ((size_t)b * a.HW + pix) * C) + l16;
#pragma unroll
            for (int j = 0; j < NW; ++j) { const u32x2_t u = q[j * 16]; v[p][j] = f32x4_t{__uint_as_float(u.x), __uint_as_float(u.y), 0.f, 0.f}; }
        } else {
            const FISE_AS1 f32x4_t* q = (const FISE_AS1 f32x4_t*)((const float*)a.x + ((size_t)b * a.Ma + i_row) * C) + l16;
#pragma unroll
            for (int j = 0; j < NW; ++j) v[p][j] = q[j * 16];
        }
    }
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        gam[j] = ((const FISE_AS1 u32x2_t*)a.gamma)[j * 16 + l16];
        bet[j] = ((const FISE_AS1 u32x2_t*)a.beta)[j * 16 + l16];
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- this wave's stage of the weights: slot p of row r holds segment p ^ ((r >> 1) & 7)
    {
        const unsigned seg = (unsigned)((lane & 7) ^ (lane >> 4)) * 16u, vd = (unsigned)(lane >> 3) * (2u * C);
        const __amdgpu_buffer_rsrc_t rs = buf(a.wq, 2u * C * C);
#pragma unroll
        for (int p = 0; p < D / 8; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (FISE_AS3 void*)(mine + p * 1024), 16, vd + (p & 1 ? seg ^ 64u : seg), (unsigned)((h * D + p * 8) * (2 * C) + wave * 128), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- LayerNorm
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int quad = p * NW + wave, row = quad * 4 + lq;
        if (quad >= QUADS) continue;
        f32x4_t x[NW];
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            x[j] = v[p][j];
            if constexpr (MAP) {
                const unsigned w0 = __float_as_uint(v[p][j].x), w1 = __float_as_uint(v[p][j].y);
                x[j] = f32x4_t{lo16(w0), hi16(w0), lo16(w1), hi16(w1)};
            }
        }
        layer_norm<16>(x, gam, bet, a.eps);
        put_row<16>(lds + row * PITCH, row, l16, x);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- this wave's 64 channels of the product (past the last row of the weights: the last eight again)
    {
        f32x4_t acc[U][2];
        bf16x8_t fw[2][U], fx[2][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = u * 16 + (u * 16 + 16 <= D ? l16 : l16 & 7);
                fw[ks][u] = *reinterpret_cast<const bf16x8_t*>(mine + r * 128 + (((lq + 4 * ks) ^ ((r >> 1) & 7)) * 16));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) fx[ks][i] = *reinterpret_cast<const bf16x8_t*>(lds + (i * 16 + l16) * PITCH + wave * 128 + (((lq + 4 * ks) ^ ((l16 >> 1) & 7)) * 16));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                acc[u][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[0][u], fx[0][i], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                acc[u][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[1][u], fx[1][i], acc[u][i], 0, 0, 0);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i) *reinterpret_cast<f32x4_t*>(mine + ((u * 2 + i) * 64 + lane) * 16) = acc[u][i];
    }
    // ---- keys and values of the two waves that go on, under the sums (keys that do not exist are zeros)
    u32x4_t k16[NT][T::QC], v16[U][2]; u32x2_t v8[U];
    const int tile = wave - (NW - 2);                          // their row tile
    if (tile >= 0) {
        const __amdgpu_buffer_rsrc_t rk = buf(a.K + (size_t)b * a.n_ctx * C, (unsigned)(a.n_ctx * C) * 2u), rv = buf(a.Vt + (size_t)b * C * a.n_stride, (unsigned)(C * a.n_stride) * 2u);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int key = t < NT - 1 ? 32 * (t >> 1) + 8 * (l16 >> 2) + 4 * (t & 1) + (l16 & 3) : 64 + l16;
#pragma unroll
            for (int c = 0; c < T::QC; ++c)
                k16[t][c] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rk, key < a.n_ctx && c * 32 + lq * 8 < D ? (unsigned)((key * C + h * D + c * 32 + lq * 8) * 2) : OOB, 0, 0));
        }
#pragma unroll
        for (int dt = 0; dt < U; ++dt) {
            const int d = dt * 16 + l16;
            const unsigned off = (unsigned)((h * D + d) * a.n_stride) * 2u;
#pragma unroll
            for (int p = 0; p < 2; ++p) v16[dt][p] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rv, d < D && 32 * p + 8 * lq < a.n_ctx ? off + (unsigned)(64 * p + 16 * lq) : OOB, 0, 0));
            v8[dt] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rv, d < D && 64 + 4 * lq < a.n_ctx ? off + (unsigned)(128 + 8 * lq) : OOB, 0, 0));
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // ---- queries: a wave sums a tile of 16 channels x 16 rows in wave order; channels past the head dim are zeros
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int id = e * NW + wave;
        if (id >= 2 * T::QC * 2) continue;
        const int u = id >> 1, i = id & 1;
        f32x4_t s = {0.f, 0.f, 0.f, 0.f};
        if (u < U)
#pragma unroll
            for (int o = 0; o < NW; ++o) s += *reinterpret_cast<const f32x4_t*>(regions + o * T::REGION + (id * 64 + lane) * 16);
        if (u * 16 + lq * 4 >= D) s = f32x4_t{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<u32x2_t*>(lds + (i * 16 + l16) * T::QPITCH + (u * 16 + lq * 4) * 2) = u32x2_t{f2bf2(s[0], s[1]), f2bf2(s[2], s[3])};
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (tile < 0) return;

    // ---- attention: lane = row l16 of the tile, keys 32 p + 8 lq + 0 .. 7 and 64 + 4 lq + 0 .. 3
    bf16x8_t q[T::QC];
#pragma unroll
    for (int c = 0; c < T::QC; ++c) q[c] = *reinterpret_cast<const bf16x8_t*>(lds + (tile * 16 + l16) * T::QPITCH + c * 64 + lq * 16);
    f32x4_t s[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        s[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < T::QC; ++c) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, k16[t][c]), q[c], s[t], 0, 0, 0);
    }
    const KeyWeights kw = key_weights(s, a.n_ctx, lq, g.scale_log2e);
    auto live = [&](unsigned x, int key) { return key + 1 < a.n_ctx ? x : key < a.n_ctx ? x & 0xffffu : 0u; };       // a word of two keys
    const int m = m0 + tile * 16 + l16;
    bf16_t* const out = (bf16_t*)a.out + ((size_t)b * a.Ma + m) * C + h * D + lq * 4;
#pragma unroll
    for (int dt = 0; dt < U; ++dt) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v16[dt][0][e] = live(v16[dt][0][e], 8 * lq + 2 * e); v16[dt][1][e] = live(v16[dt][1][e], 32 + 8 * lq + 2 * e); }
        const u32x4_t tail = {live(v8[dt].x, 64 + 4 * lq), live(v8[dt].y, 66 + 4 * lq), 0, 0};
        const f32x4_t x = weighted(v16[dt][0], v16[dt][1], tail, kw);
        if (m < a.Ma && dt * 16 + lq * 4 < D) *(FISE_AS1 u32x2_t*)(out + dt * 16) = u32x2_t{f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
    }
#endif
}

template <bool MAP> static int launch(const CrossDev& g, hipStream_t st) {
    constexpr int lds = 32 * 2 * CROSS_C + CROSS_HEADS * 3 * (CROSS_C / CROSS_HEADS) * 128 + 32 * 4;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&cross_attention_kernel<MAP>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "cross attention: cannot raise the dynamic LDS limit");
    const CrossArgs& a = g.a;
    {
        const double rows = (double)a.B * a.Ma, el = MAP ? 2.0 : 4.0;
        ProfileScope prof(PROF_ROWS_GEMM, rows * CROSS_C * 4.0 * (CROSS_C + a.n_ctx), 4.0 * CROSS_C * (CROSS_C + (double)a.B * a.n_ctx) + 2 * el * rows * CROSS_C, st);
        hipLaunchKernelGGL((cross_attention_kernel<MAP>), dim3((unsigned)(g.gx * a.B)), dim3(512), lds, st, g);
    }
    FISE_CHECK_LAUNCH("cross attention");
    return FISE_OK;
}

template <int C, bool MAP> static int launch_query(const CrossDev& g, hipStream_t st) {
    constexpr int lds = QueryTile<C>::LDS;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&query_attention_kernel<C, MAP>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "query attention: cannot raise the dynamic LDS limit");
    const CrossArgs& a = g.a;
    {
        const double rows = (double)a.B * a.Ma, el = MAP ? 2.0 : 4.0;
        ProfileScope prof(PROF_ROWS_GEMM, rows * C * (2.0 * C + 4.0 * a.n_ctx), 2.0 * C * (C + 2.0 * a.B * a.n_ctx) + (el + 2.0) * rows * C, st);
        hipLaunchKernelGGL((query_attention_kernel<C, MAP>), dim3((unsigned)(g.gx * a.B * CROSS_HEADS)), dim3(C), lds, st, g);
    }
    FISE_CHECK_LAUNCH("query attention");
    return FISE_OK;
}

static CrossDev device_args(const CrossArgs& a, int C) {
    CrossDev g{};
    g.a = a;
    g.gx = ceil_div(a.Ma, 32); g.scale_log2e = 1.4426950408889634f / sqrtf((float)(C / CROSS_HEADS));
    g.d_gx = fast_div(g.gx); g.d_tiles = fast_div(g.gx * a.B);
    if (a.tile_idx) { g.d_tt = fast_div(a.tile * a.tile); g.d_tile = fast_div(a.tile); g.d_tiles_w = fast_div(a.tiles_w); }
    return g;
}

int launch_cross(const CrossArgs& a, hipStream_t st) {
    const CrossDev g = device_args(a, CROSS_C);
    return a.tile_idx ? launch<true>(g, st) : launch<false>(g, st);
}

int launch_query_attention(const CrossArgs& a, int C, hipStream_t st) {
    const CrossDev g = device_args(a, C);
    if (C == 320) return a.tile_idx ? launch_query<320, true>(g, st) : launch_query<320, false>(g, st);
    return a.tile_idx ? launch_query<640, true>(g, st) : launch_query<640, false>(g, st);
}

}  // namespace fise
