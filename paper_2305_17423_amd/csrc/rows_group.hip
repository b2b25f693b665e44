// Several products of the same compact rows as one launch: out_g[m, n] = sum_k x[m, k] w_g[n, k] for every product g of a group, as compact rows or with
// its columns as rows (keys and transposed values of a prompt for all cross-attention layers).
//  - A workgroup owns up to 224 rows and seven units of 16 columns; the units of all products stand one behind the other, so a tile may end one
//    product and begin the next.  24960 columns of 16 blocks are 223 tiles: one round of the CUs, every weight passes the LDS once.
//  - Stages of 64 channels of both operands go through one ring by LDS-direct loads, pieces of eight rows of 128 bytes, each with the
//    descriptor of its product.  Four waves: two share K (32 of a stage's 64 channels), two the rows; 16 x 16 x 32 products.
//  - The two K halves of a result meet in LDS: one wave finishes the first four units, the other the last three.
// Bound by what the CUs get through LDS-direct loads (417 KB a tile of 160 rows x 768 channels) and the weights from memory (38 MB, 7.4 us at the rate of a
// large copy).  Tiles of 64 x 64 are 1170 for the same, 230 MB through the LDS.  24960 columns of 768 channels, us, those and now: 8 rows 12.0, 10.5; 96 rows
// 17.8, 12.8; 154 rows 24.0, 15.5; 200 rows 25.6, 19.5; 308 rows 35.2, 27.8; 616 rows 62.3, 49.0.
#include <algorithm>
#include <type_traits>
#include "igemm.h"
#include "profile.h"

namespace fise {

struct RowsGroup {
    const bf16_t* x;
    int rows, K, Ma, stride, units, gx;      // Ma: rows of a batch element; stride: of a transposed column
    FastDiv d_gx, d_Ma;
    GemmGroup g;                             // first: in units of 16 columns
};

template <int RT> struct GroupTile {
    static constexpr int BM = 32 * RT, CT = GROUP_UNITS, STAGE = (BM + 16 * CT) * 128, NS = RT == 7 ? 3 : RT == 5 ? 4 : RT == 3 ? 5 : 6, LDS = NS * STAGE + 1024;      // and a place for loads of nothing
};

template <int RT>
__global__ __launch_bounds__(256, 1) void rows_group_kernel(const RowsGroup a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = GroupTile<RT>;
    constexpr int BM = T::BM, NS = T::NS, CT = T::CT, C0 = (CT + 1) / 2, WL = (2 * CT + 3) / 4;       // WL: weight loads of a lane and stage
    constexpr unsigned OOB = 0x80000000u;
    static_assert(4 * C0 * RT * 1024 <= NS * T::STAGE, "hand-over");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    asm volatile("" ::"s"(a.x), "s"(a.rows), "s"(a.K), "s"(a.Ma), "s"(a.stride), "s"(a.units), "s"(a.gx), "s"(a.d_gx.mul), "s"(a.d_Ma.mul));
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4, l8 = lane >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kh = wave & 1, mw = wave >> 1;
    const int first = lane < GEMM_GROUP ? a.g.first[lane] : 1 << 30;
    // every XCD gets a contiguous run of (columns, rows), rows fastest
    const int run = (int)gridDim.x >> 3;
    int w = blockIdx.x;
    if (w < (run << 3)) w = (w & 7) * run + (w >> 3);
    const int cg = (int)fdiv((unsigned)w, a.d_gx), m0 = (w - cg * a.gx) * BM, u0 = cg * CT;

    // ---- stages: wave v loads the pieces v, v + 4 ... of x and of the weights; 16-byte segments swizzled with (row >> 1) & 7
    const unsigned pitch = (unsigned)a.K * 2u;
    unsigned va[RT], vb[WL], wbytes[WL]; const bf16_t* wp[WL];
#pragma unroll
    for (int l = 0; l < RT; ++l) {
        const int r = (wave + 4 * l) * 8 + l8;
        va[l] = m0 + r < a.rows ? (unsigned)(m0 + r) * pitch + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16) : OOB;
    }
#pragma unroll
    for (int l = 0; l < WL; ++l) {
        const int piece = wave + 4 * l, u = u0 + (piece >> 1), g = __popcll(__ballot(u >= first)) - 1, r = (piece & 1) * 8 + l8;
        const bool live = piece < 2 * CT && u < a.units;
        wp[l] = a.g.w[g];
        wbytes[l] = live ? (unsigned)a.g.N[g] * pitch : 0u;
        vb[l] = (unsigned)((u - a.g.first[g]) * 16 + r) * pitch + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
    }
    const int steps = a.K >> 6;
    const unsigned xbytes = (unsigned)a.rows * pitch;
    int issued = 0; unsigned slot = 0;
    auto issue = [&]() {                                 // past the last stage: descriptors of size zero, no traffic
        unsigned char* const base = lds + slot;
        const unsigned soff = (unsigned)issued * 128u;
#pragma unroll
        for (int l = 0; l < WL; ++l) {
            const __amdgpu_buffer_rsrc_t rw = buf(wp[l], issued < steps ? wbytes[l] : 0u);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (FISE_AS3 void*)(wave + 4 * l < 2 * CT ? base + (BM + (wave + 4 * l) * 8) * 128 : lds + NS * T::STAGE), 16, vb[l], soff, 0, 0);
        }
        const __amdgpu_buffer_rsrc_t rx = buf(a.x, issued < steps ? xbytes : 0u);
#pragma unroll
        for (int l = 0; l < RT; ++l) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (FISE_AS3 void*)(base + (wave + 4 * l) * 1024), 16, va[l], soff, 0, 0);
        ++issued;
        slot = slot == (NS - 1) * T::STAGE ? 0u : slot + T::STAGE;
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue();
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
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * (RT + WL)) : "memory");
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

    // ---- the K halves: each wave hands over the units that it does not finish (a branch per half: indexed by it the sums would go through memory)
    f32x4_t* const hand = reinterpret_cast<f32x4_t*>(lds);
    auto give = [&](auto from, auto n) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < decltype(n)::value; ++j) hand[((wave * RT + i) * C0 + j) * 64 + lane] = acc[i][decltype(from)::value + j];
    };
    auto finish = [&](auto from, auto n) {
#pragma unroll
        for (int j = 0; j < decltype(n)::value; ++j) {
            const int u = u0 + decltype(from)::value + j, g = __popcll(__ballot(u >= first)) - 1;
            if (u >= a.units) break;
            const int N = a.g.N[g], col = (u - a.g.first[g]) * 16 + lq * 4;
            bf16_t* const out = a.g.out[g];
            const bool tokens = a.g.mode[g] == OUT_TOKENS_T;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int m = m0 + (mw * RT + i) * 16 + l16;
                const f32x4_t y = acc[i][decltype(from)::value + j] + hand[(((wave ^ 1) * RT + i) * C0 + j) * 64 + lane];
                const u32x2_t packed = {f2bf2(y[0], y[1]), f2bf2(y[2], y[3])};
                if (m >= a.rows) continue;
                if (tokens) {
                    const unsigned b = fdiv((unsigned)m, a.d_Ma);
                    FISE_AS1 bf16_t* const p = (FISE_AS1 bf16_t*)(out + ((size_t)b * N + col) * a.stride + (m - (int)b * a.Ma));
#pragma unroll
                    for (int q = 0; q < 4; ++q) p[(size_t)q * a.stride] = (bf16_t)(q & 1 ? packed[q >> 1] >> 16 : packed[q >> 1]);
                } else {
                    *(FISE_AS1 u32x2_t*)(out + (size_t)m * N + col) = packed;
                }
            }
        }
    };
    using Zero = std::integral_constant<int, 0>; using Low = std::integral_constant<int, C0>; using High = std::integral_constant<int, CT - C0>;
    if (kh) give(Zero(), Low()); else give(Low(), High());
    __syncthreads();
    if (kh) finish(Low(), High()); else finish(Zero(), Low());
#endif
}

template <int RT>
static int launch_rows(const RowsGroup& a, int cols, hipStream_t st) {
    constexpr int lds = GroupTile<RT>::LDS;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&rows_group_kernel<RT>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "rows group: cannot raise the dynamic LDS limit");
    {
        ProfileScope prof(PROF_ROWS_GEMM, 2.0 * a.rows * cols * (double)a.K, 2.0 * ((double)cols * a.K + (double)a.rows * a.K + (double)a.rows * cols), st);
        hipLaunchKernelGGL((rows_group_kernel<RT>), dim3((unsigned)(a.gx * ceil_div(a.units, GROUP_UNITS))), dim3(256), lds, st, a);
    }
    FISE_CHECK_LAUNCH("rows group");
    return FISE_OK;
}

// Compact rows and token columns of a buffer without a tile list; sizes are the grouped launch's (32-bit offsets into rows and weights).
bool rows_group_takes(const IgemmArgs& a, const GemmProduct* p, int n) {
    int cols = 0;
    for (int i = 0; i < n; ++i) {
        if (p[i].mode != OUT_COMPACT && p[i].mode != OUT_TOKENS_T) return false;
        cols += p[i].N;
    }
    return !a.tile_idx && a.Ho == 1 && a.ksize == 1 && a.C1 == 0 && a.K == a.C0 && a.K % 64 == 0 && group_tile(a.B * a.Ma, cols, a.Ma % 4 == 0) > 0;
}

int launch_rows_group(const IgemmArgs& b, const GemmProduct* p, int n, hipStream_t st) {
    RowsGroup a{};
    a.x = b.a0; a.rows = b.B * b.Ma; a.K = b.K; a.Ma = b.Ma; a.stride = b.Wo;
    for (int i = 0; i < GEMM_GROUP; ++i) {
        a.g.first[i] = i < n ? a.units : 1 << 30;
        if (i >= n) continue;
        a.g.w[i] = p[i].w; a.g.out[i] = p[i].out; a.g.N[i] = p[i].N; a.g.mode[i] = p[i].mode;
        a.units += p[i].N / 16;
    }
    const int rt = group_tile(a.rows, a.units * 16, a.Ma % 4 == 0);
    a.gx = ceil_div(a.rows, 32 * rt); a.d_gx = fast_div(a.gx); a.d_Ma = fast_div(a.Ma);
    const int cols = a.units * 16;
    return rt == 1 ? launch_rows<1>(a, cols, st) : rt == 2 ? launch_rows<2>(a, cols, st) : rt == 3 ? launch_rows<3>(a, cols, st) : rt == 5 ? launch_rows<5>(a, cols, st) : launch_rows<7>(a, cols, st);
}

}  // namespace fise
