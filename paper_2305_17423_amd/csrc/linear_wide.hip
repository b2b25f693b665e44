// Linears of many compact rows into float rows (attention output and feed-forward projections, residual added):
//   out[m, n] = sum_k x[m, k] w[n, k] + bias[n] + res[m, n]
// on tiles of 64 or 128 rows x 80 columns.  What a CU gets through LDS-direct loads (71 - 88 GB/s) bounds them, so the bytes per product decide:
// a stage of 64 channels brings 26 KB for 128 x 80 outputs, where tiles of 64 x 128 bring 24 KB for fewer; and 80 columns divide widths of
// 320, 640 and 1280 without a remainder, so 8192 x 320 and 2048 x 640 outputs are one tile for each of the 256 CUs.
//  - Four waves: two share K (32 of a stage's 64 channels each), two the rows; 16 x 16 x 32 products.
//  - Residual and bias are requested in front of the K loop.
//  - The two K halves of a row meet in LDS, each finishing half of the row tiles.
//  - Every XCD gets a contiguous run of tiles, columns fastest: a row of x is read by one L2.
#include <algorithm>
#include "igemm.h"
#include "profile.h"

namespace fise {

struct LinearWide {
    const bf16_t *x, *w, *bias;
    const float* res;
    float* out;
    bf16_t* mirror;                  // bf16 copy of the rows, or null
    int rows, N, K, gy;
    FastDiv d_gy;
    unsigned bias_bytes, res_bytes;
};

template <int RT> struct LinearTile {
    static constexpr int BM = 32 * RT, STAGE = (BM + 80) * 128, NS = 4, LDS = NS * STAGE + 1024;      // and a place for loads of nothing
};

template <int RT>
__global__ __launch_bounds__(256, 1) void linear_wide_kernel(const LinearWide a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = LinearTile<RT>;
    constexpr int BM = T::BM, NS = T::NS, CT = 5, HT = RT / 2;
    constexpr unsigned OOB = 0x80000000u;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    asm volatile("" ::"s"(a.x), "s"(a.w), "s"(a.bias), "s"(a.res), "s"(a.out), "s"(a.mirror), "s"(a.rows), "s"(a.N), "s"(a.K), "s"(a.gy), "s"(a.d_gy.mul), "s"(a.bias_bytes), "s"(a.res_bytes));
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4, l8 = lane >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kh = wave & 1, mw = wave >> 1;
    const int run = (int)gridDim.x >> 3;
    int u = blockIdx.x;
    if (u < (run << 3)) u = (u & 7) * run + (u >> 3);
    const int bx = (int)fdiv((unsigned)u, a.d_gy), by = u - bx * a.gy, m0 = bx * BM, n0 = by * 80;

    // ---- stages: pieces of eight rows of 128 bytes, wave v loads the pieces v, v + 4 ... of x and of w; segments swizzled with (row >> 1) & 7
    const unsigned pitch = (unsigned)a.K * 2u;
    unsigned va[RT], vb[3];
#pragma unroll
    for (int l = 0; l < RT; ++l) {
        const int r = (wave + 4 * l) * 8 + l8;
        va[l] = m0 + r < a.rows ? (unsigned)(m0 + r) * pitch + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16) : OOB;
    }
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const int r = (wave + 4 * l) * 8 + l8;
        vb[l] = r < 80 ? (unsigned)(n0 + r) * pitch + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16) : OOB;
    }
    const int steps = a.K >> 6;
    const unsigned xbytes = (unsigned)a.rows * pitch, wbytes = (unsigned)a.N * pitch;
    int issued = 0; unsigned slot = 0;
    auto issue = [&]() {                                 // past the last stage: descriptors of size zero, no traffic
        const __amdgpu_buffer_rsrc_t rx = buf(a.x, issued < steps ? xbytes : 0u), rw = buf(a.w, issued < steps ? wbytes : 0u);
        unsigned char* const base = lds + slot;
        const unsigned soff = (unsigned)issued * 128u;
#pragma unroll
        for (int l = 0; l < 3; ++l)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (FISE_AS3 void*)(wave + 4 * l < 10 ? base + (BM + (wave + 4 * l) * 8) * 128 : lds + NS * T::STAGE), 16, vb[l], soff, 0, 0);
#pragma unroll
        for (int l = 0; l < RT; ++l) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (FISE_AS3 void*)(base + (wave + 4 * l) * 1024), 16, va[l], soff, 0, 0);
        ++issued;
        slot = slot == (NS - 1) * T::STAGE ? 0u : slot + T::STAGE;
    };
    issue();
    // ---- what the epilogue adds, ahead of the other stages
    u32x2_t e_bias[CT]; f32x4_t e_res[HT][CT];
    {
        const __amdgpu_buffer_rsrc_t sb = buf(a.bias, a.bias_bytes), sr = buf(a.res, a.res_bytes);
#pragma unroll
        for (int c = 0; c < CT; ++c) e_bias[c] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(sb, (unsigned)(n0 + c * 16 + lq * 4) * 2u, 0, 0));
#pragma unroll
        for (int i = 0; i < HT; ++i) {
            const int m = m0 + (mw * RT + kh * HT + i) * 16 + l16;
#pragma unroll
            for (int c = 0; c < CT; ++c)
                e_res[i][c] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(sr, m < a.rows ? ((unsigned)m * (unsigned)a.N + (unsigned)(n0 + c * 16 + lq * 4)) * 4u : OOB, 0, 0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 1; s < NS - 1; ++s) issue();
    __builtin_amdgcn_sched_barrier(0);

    f32x4_t acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[i][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const unsigned rd = (unsigned)(l16 * 128 + (((kh * 4 + lq) ^ ((l16 >> 1) & 7)) * 16));      // an operand within 16 rows
    unsigned rs = 0;
#pragma unroll 1
    for (int k = 0; k < steps; ++k) {
        // the loads of this stage are the oldest; behind the barrier every wave has the stage before it in registers
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * (RT + 3)) : "memory");
        bf16x8_t fa[RT], fb[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) fb[c] = *reinterpret_cast<const bf16x8_t*>(lds + rs + BM * 128 + rd + c * 2048);
#pragma unroll
        for (int i = 0; i < RT; ++i) fa[i] = *reinterpret_cast<const bf16x8_t*>(lds + rs + (mw * RT + i) * 2048 + rd);
        rs = rs == (NS - 1) * T::STAGE ? 0u : rs + T::STAGE;
        __builtin_amdgcn_sched_barrier(0);
        issue();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < RT; ++i) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[c], fa[i], acc[i][c], 0, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- the K halves: each wave finishes half of its row tiles and hands over the others
    f32x4_t* const hand = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) hand[((wave * HT + i) * CT + c) * 64 + lane] = kh ? acc[i][c] : acc[HT + i][c];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HT; ++i) {
        const int m = m0 + (mw * RT + kh * HT + i) * 16 + l16;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            f32x4_t y = (kh ? acc[HT + i][c] : acc[i][c]) + hand[(((wave ^ 1) * HT + i) * CT + c) * 64 + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                y[q] += q & 1 ? hi16(e_bias[c][q >> 1]) : lo16(e_bias[c][q >> 1]);
                y[q] += e_res[i][c][q];
            }
            if (m < a.rows) {
                const size_t o = (size_t)m * a.N + n0 + c * 16 + lq * 4;
                *(FISE_AS1 f32x4_t*)(a.out + o) = y;
                if (a.mirror) *(FISE_AS1 u32x2_t*)(a.mirror + o) = u32x2_t{f2bf2(y[0], y[1]), f2bf2(y[2], y[3])};
            }
        }
    }
#endif
}

template <int RT>
static int launch_lw(const LinearWide& a, hipStream_t st) {
    constexpr int lds = LinearTile<RT>::LDS;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&linear_wide_kernel<RT>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "linear: cannot raise the dynamic LDS limit");
    {
        ProfileScope prof(PROF_IGEMM_WIDE, 2.0 * a.rows * a.N * (double)a.K, 2.0 * ((double)a.N * a.K + (double)a.rows * a.K) + 8.0 * a.rows * a.N, st);
        hipLaunchKernelGGL((linear_wide_kernel<RT>), dim3((unsigned)(ceil_div(a.rows, 32 * RT) * a.gy)), dim3(256), lds, st, a);
    }
    FISE_CHECK_LAUNCH("linear");
    return FISE_OK;
}

bool linear_wide_takes(const IgemmArgs& a) {
    const long long rows = (long long)a.B * a.Ma, lim = 1ll << 31;
    return a.a_compact && a.ksize == 1 && a.C1 == 0 && a.K == a.C0 && a.K % 64 == 0 && a.N % 80 == 0 && a.K2 == 0 && a.pro == PRO_NONE && a.nsect == 1 && !a.geglu &&
           a.out_mode[0] == OUT_COMPACT_F32 && (!a.res || a.res_compact == 2) && !a.temb && !a.bias2 && !a.nview && !a.ln_out &&
           rows * std::max(a.K * 2ll, a.N * 4ll) < lim && (long long)a.N * a.K * 2 < lim && rows < 1 << 24 && linear_tile((int)rows, a.N) > 0;
}

int launch_linear_wide(const IgemmArgs& g, hipStream_t st) {
    LinearWide a{};
    a.x = (const bf16_t*)g.a0; a.w = (const bf16_t*)g.w; a.bias = (const bf16_t*)g.bias; a.res = (const float*)g.res; a.out = (float*)g.out[0]; a.mirror = g.mirror;
    a.rows = g.B * g.Ma; a.N = g.N; a.K = g.K; a.gy = g.N / 80; a.d_gy = fast_div(a.gy);
    a.bias_bytes = g.bias ? (unsigned)g.N * 2u : 0u; a.res_bytes = g.res ? (unsigned)a.rows * (unsigned)g.N * 4u : 0u;
    return linear_tile(a.rows, a.N) == 4 ? launch_lw<4>(a, st) : launch_lw<2>(a, st);
}

}  // namespace fise
