// Normalisation and the product behind it as one launch:
//
//   out[row, n] = epilogue( sum_k N(x[row])[k] * W[n, k] ),   N = LayerNorm of the row, or GroupNorm with given statistics
//
// the query / key / value products, the cross-attention queries and the first feed-forward product (GEGLU gate) of a transformer
// block, and its input product where no normalised copy of the map is kept.  Widths 320, 640 and 1280.
//  - A workgroup of eight waves normalises its 16*RT rows once, straight from the float residual stream (or the map) into LDS as bf16:
//    20 - 90 KB, all of K.  No launch writes normalised rows and no launch reads them back.
//  - Every wave owns 16*CT columns at a time and streams their weights through an LDS ring of its own (LDS-direct loads, eight rows of 128 bytes
//    each, ND stages of 64 channels): behind the barrier of the rows there is none.  The ring runs on over the end of a column
//    tile, so the next tile's weights travel under the epilogue.
//  - Where the rows come from is part of the kernel's type, the touched lines are a fixed number of loads and the bias waits in LDS: the
//    compiler then counts the loads in flight exactly.  With a run-time source, a loop of touches and the bias in registers it waited for every load,
//    the first stages of cold weights among them, in front of the normalisation and of each column tile (rows normalised after 4.2 us of an 8 us launch,
//    7.2 of 15 with GEGLU at 96 rows): steps of 12 of 64 and 43 of 144 tiles 2277 -> 2250 and 4226 -> 4174 us, dense pass 5047 -> 4975.
//  - 16 x 16 x 32 products: a lane ends up with four consecutive columns of a row, or, with the operands exchanged, four consecutive
//    rows of a column (the transposed values); results go from registers to memory, there is no sum over waves.
// Bound by the LDS (operands of both sides, 2 RT + 4 CT KB a wave and stage) and the rate of LDS-direct loads for many rows, by its start, the rows and the
// first weights (5 - 6 us) for few.  Against a LayerNorm launch and the gathered GEMM (us): GEGLU 1536 x 2560 x 320 18 -> 9, 8192 x 2560 x
// 320 60 -> 24, 2048 x 5120 x 640 44 -> 27, 96 x 10240 x 1280 20 -> 16; queries, keys and values 1536 x 960 x 320 13.5 -> 7.8, 96 x 3840 x
// 1280 13.5 -> 11.3; one product 1536 x 320 x 320 8 -> 5.7, 24 x 1280 x 1280 10 -> 8.1.  Weights straight into matrix registers (16 rows of 64 bytes a load, no
// LDS) were up to 1.6 times slower from 100 KB of weights a workgroup on: 37 GB/s per CU instead of 60.
#include <algorithm>
#include "igemm.h"
#include "profile.h"

namespace fise {

struct NormGemmDev {
    NormGemmArgs a;
    int gx, per, units, t_tokens, trans4, pixels, touch, ks;
    FastDiv d_gx, d_Ma, d_tt, d_tile, d_tiles_w, d_cpg;
};

// LDS of a workgroup: rows of K bf16 whose 16-byte segments are XOR-swizzled with (row >> 1) & 7, at a pitch of 128 bytes modulo 256,
// so that sixteen rows' operand reads meet no bank twice; then the rows' positions; then (GroupNorm) the scale / shift table.
template <int KM> constexpr int ng_pitch() { return 640 * KM + (KM == 1 ? 0 : 128); }

template <int KM, int RT, int CT, int ND, bool GEGLU, int SRC>
__global__ __launch_bounds__(64 * NG_WAVES, 2) void norm_gemm_kernel(const NormGemmDev g) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int NW = NG_WAVES, K = 320 * KM, BM = 16 * RT, PITCH = ng_pitch<KM>(), LPR = 16 * KM, RPW = 64 / LPR, P = BM / (NW * RPW);
    constexpr int OC = GEGLU ? 16 : 16 * CT, NK = 5 * KM;      // output columns of a unit, stages of 64 channels
    constexpr unsigned OOB = 0x80000000u;                 // beyond every descriptor: no traffic
    constexpr int NG_TOUCH = 2;                           // lines a lane touches at most
    static_assert(P >= 1 && BM % (NW * RPW) == 0 && (!GEGLU || CT == 2), "rows per wave");
    const NormGemmArgs& a = g.a;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    int2* const rowpos = reinterpret_cast<int2*>(lds + BM * PITCH);
    constexpr int WST = CT * 2048;                        // bytes of a stage of weights in LDS
    unsigned char* const wring = lds + BM * PITCH + BM * 8;
    constexpr bool BIAS = norm_gemm_has_bias(GEGLU, SRC);
    unsigned char* const lbias = wring + NW * ND * WST;
    float2* const table = reinterpret_cast<float2*>(lbias + (BIAS ? NG_BIAS : 0));
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive workgroups go round-robin to the 8 XCDs: each gets a contiguous run of (columns, rows), rows fastest
    const int total = gridDim.x, chunk = total >> 3;
    int w = blockIdx.x;
    if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
    const int cs = (int)fdiv((unsigned)w, g.d_gx), bx = w - cs * g.gx;
    const int rows = a.B * a.Ma, m0 = bx * BM;
    const int t0 = cs * g.per, t1 = min(g.units, t0 + g.per);

    // ---- rows: LPR lanes a row, five pieces of four channels each, all rows of the wave requested together
    const int l = lane % LPR;
    f32x4_t v[P][5];
    const int b_first = (int)fdiv((unsigned)m0, g.d_Ma);
    unsigned rb[P], rm[P], rt[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const unsigned gm = (unsigned)min(m0 + p * (NW * RPW) + wave * RPW + lane / LPR, rows - 1);
        rb[p] = fdiv(gm, g.d_Ma); rm[p] = gm - rb[p] * (unsigned)a.Ma; rt[p] = 0;
    }
    if (g.pixels)
#pragma unroll
        for (int p = 0; p < P; ++p) rt[p] = (unsigned)((const FISE_AS1 int*)a.tile_idx)[fdiv(rm[p], g.d_tt)];
    if constexpr (SRC == NG_ROWS_LN)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const FISE_AS1 f32x4_t* q = (const FISE_AS1 f32x4_t*)((const float*)a.x + (size_t)(rb[p] * (unsigned)a.Ma + rm[p]) * K) + l;
#pragma unroll
            for (int j = 0; j < 5; ++j) v[p][j] = q[j * LPR];
        }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (g.pixels) {                                  // position on the map, from here on in place of the row
            const unsigned rp = rm[p] - fdiv(rm[p], g.d_tt) * (unsigned)(a.tile * a.tile), py = fdiv(rp, g.d_tile), ty = fdiv(rt[p], g.d_tiles_w);
            rm[p] = (ty * a.tile + py) * (unsigned)a.Wo + (rt[p] - ty * a.tiles_w) * a.tile + (rp - py * a.tile);
        }
        if (l == 0) rowpos[p * (NW * RPW) + wave * RPW + lane / LPR] = make_int2((int)rb[p], (int)rm[p]);
    }
    if constexpr (SRC != NG_ROWS_LN)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const FISE_AS1 u32x2_t* q = (const FISE_AS1 u32x2_t*)((const bf16_t*)a.x + ((size_t)rb[p] * (a.Ho * a.Wo) + rm[p]) * K) + l;
#pragma unroll
            for (int j = 0; j < 5; ++j) { const u32x2_t u = q[j * LPR]; v[p][j] = f32x4_t{__uint_as_float(u.x), __uint_as_float(u.y), 0.f, 0.f}; }
        }
    u32x2_t gam[5], bet[5];
    if constexpr (SRC == NG_ROWS_LN || SRC == NG_MAP_LN)
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            gam[j] = ((const FISE_AS1 u32x2_t*)a.gamma)[j * LPR + l];
            bet[j] = ((const FISE_AS1 u32x2_t*)a.beta)[j * LPR + l];
        }
    __builtin_amdgcn_sched_barrier(0);

    // Where a workgroup has at most four units the waves also split K: 2^ks of them a unit, part `part` of its stages each.
    const int part = wave & ((1 << g.ks) - 1), step = NW >> g.ks;
    const int per_k = (NK + (1 << g.ks) - 1) >> g.ks, k0 = min(NK, part * per_k), kn = min(NK, k0 + per_k) - k0;
    // ---- weights: unit t is 16*CT weight rows (GEGLU: 16 of the values, 16 of the gates N further down)
    const bf16_t* wp = nullptr; unsigned wbytes = 0, wrow = 0;
    auto set_unit = [&](int t) {                          // past the range: a descriptor of size zero, no traffic
        const int col = t * OC, s = GEGLU ? 0 : (col >= a.sect_n) + (col >= 2 * a.sect_n);
        wp = s == 0 ? a.w[0] : s == 1 ? a.w[1] : a.w[2];
        wbytes = t < t1 ? (unsigned)((GEGLU ? 2 * a.N : a.sect_n) * (2 * K)) : 0u;
        wrow = (unsigned)(col - s * a.sect_n) * (2u * K) + k0 * 128u;
    };
    // LDS ring: slot p of row r holds segment p ^ ((r >> 1) & 7); a load fills eight rows
    const unsigned seg = (unsigned)((lane & 7) ^ ((lane >> 4) & 7)) * 16u;
    const unsigned vd0 = (unsigned)(lane >> 3) * (2u * K) + seg, vd1 = (unsigned)(8 + (lane >> 3)) * (2u * K) + (seg ^ 64u);
    unsigned char* const my_ring = wring + __builtin_amdgcn_readfirstlane(wave) * (ND * WST);
    auto load = [&](int u) {                              // the unit's next stage into ring slot u
        const __amdgpu_buffer_rsrc_t rs = buf(wp, wbytes);
#pragma unroll
        for (int q = 0; q < 2 * CT; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(my_ring + u * WST + q * 1024), 16,
                                                     q & 1 ? vd1 : vd0, wrow + (q < 2 ? 0u : GEGLU ? (unsigned)a.N * (2u * K) : 16u * (2u * K)), 0, 0);
        wrow += 128u;
    };
    // the bias of this workgroup's columns (GEGLU: of the values, then of the gates), 16 bytes a thread, on its way to LDS
    u32x4_t bias16 = u32x4_t{0, 0, 0, 0};
    if constexpr (BIAS) {
        const __amdgpu_buffer_rsrc_t rs = buf(a.bias, a.bias ? (unsigned)((GEGLU ? 2 : 1) * a.N) * 2u : 0u);
        const int half = g.per * OC / 8;                 // pieces of the values
        bias16 = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)(t0 * OC + (GEGLU && tid >= half ? a.N - half * 8 : 0) + tid * 8) * 2u, 0, 0));
    }
    // Row tiles that share a slice of the weights walk it in step, so each of its lines is cold for all of them at once: they first touch
    // the slice, each a share of its lines (one dword a line, into the ring before it is filled; NG_TOUCH x 512 lines a row tile at most).  512 x 10240 x 1280 38 -> 30.4 us, 96 rows
    // 18.4 -> 16.0; slices under 200 KB or two row tiles lose 0.3 - 1 us.
    {
        const int col0 = t0 * OC, s = GEGLU ? 0 : (col0 >= a.sect_n) + (col0 >= 2 * a.sect_n), n = GEGLU ? 32 * (t1 - t0) : min(t1 * OC, (s + 1) * a.sect_n) - col0;
        const __amdgpu_buffer_rsrc_t rs = buf(s == 0 ? a.w[0] : s == 1 ? a.w[1] : a.w[2], g.touch ? (unsigned)((GEGLU ? 2 * a.N : a.sect_n) * (2 * K)) : 0u);
#pragma unroll
        for (int k = 0; k < NG_TOUCH; ++k) {
            const int q = ((k * g.gx + bx) * NW + wave) * 64 + lane, r = q / NK, row = GEGLU ? (r & 1 ? a.N : 0) + col0 + (r >> 1) : col0 - s * a.sect_n + r;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)my_ring, 4, q < n * NK ? (unsigned)row * (2u * K) + (unsigned)(q - r * NK) * 128u : OOB, 0, 0, 0);
        }
    }
    int t = t0 + (wave >> g.ks);
    set_unit(t);
#pragma unroll
    for (int u = 0; u < ND; ++u) {
        if (u == kn) set_unit(t + step);
        load(u);
    }
    int slot = 0, pos = ND <= kn ? ND : ND - kn;                               // next stage to read, stages of the unit that have been requested
    __builtin_amdgcn_sched_barrier(0);

    // ---- normalise into LDS
    if constexpr (SRC == NG_MAP_GN) {                     // (scale, shift) of the tile's batch elements (two at most: Ma >= BM)
        for (int e = tid; e < 2 * K; e += 64 * NW) {
            const int bb = min(a.B - 1, b_first + (e >= K)), c = e >= K ? e - K : e, gi = bb * a.G + (int)fdiv((unsigned)c, g.d_cpg);
            const float sc = a.gn_rstd[gi] * bf2f(a.gamma[c]);
            table[e] = make_float2(sc, bf2f(a.beta[c]) - a.gn_mean[gi] * sc);
        }
        __syncthreads();
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int r = p * (NW * RPW) + wave * RPW + lane / LPR;
        f32x4_t x[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            x[j] = v[p][j];
            if constexpr (SRC != NG_ROWS_LN) {
                const unsigned w0 = __float_as_uint(v[p][j].x), w1 = __float_as_uint(v[p][j].y);
                x[j] = f32x4_t{lo16(w0), hi16(w0), lo16(w1), hi16(w1)};
            }
        }
        if constexpr (SRC == NG_MAP_GN) {
            const float2* ss = table + ((int)fdiv((unsigned)min(m0 + r, rows - 1), g.d_Ma) - b_first) * K;
#pragma unroll
            for (int j = 0; j < 5; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) { const float2 s = ss[(j * LPR + l) * 4 + q]; x[j][q] = x[j][q] * s.x + s.y; }
        } else if constexpr (SRC != NG_MAP_RAW) {
            layer_norm<LPR>(x, gam, bet, a.eps);
        }
        put_row<LPR>(lds + r * PITCH, r, l, x);
    }
    if constexpr (BIAS)
        if (tid < NG_BIAS / 16) *reinterpret_cast<u32x4_t*>(lbias + tid * 16) = bias16;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // not the loads of the weights

    // ---- column tiles
    const unsigned rd0 = (unsigned)(l16 * PITCH + ((lq ^ ((l16 >> 1) & 7)) * 16)), rd1 = rd0 ^ 64u, rw = (unsigned)(l16 * 128) + ((lq ^ ((l16 >> 1) & 7)) * 16);     // operand of channels 0 - 31 / 32 - 63 of a stage
    auto column_tile = [&](auto tokens) {
        constexpr bool TOKENS = decltype(tokens)::value;
        f32x4_t acc[RT][CT];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[i][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        const int col = t * OC, sect = GEGLU ? 0 : (col >= a.sect_n) + (col >= 2 * a.sect_n);
        const int mode = GEGLU ? OUT_COMPACT : sect == 0 ? a.mode[0] : sect == 1 ? a.mode[1] : a.mode[2];
        auto run = [&]() {
            bf16x8_t fa[2][2][RT], fb[2][2][CT];
            unsigned r0 = rd0 + k0 * 128u, r1 = rd1 + k0 * 128u;
            auto read = [&](bf16x8_t (&x)[2][RT], bf16x8_t (&w)[2][CT]) {       // the oldest stage, which has landed
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ND - 1) * 2 * CT) : "memory");
                const unsigned char* const stage = my_ring + slot * WST;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                    for (int c = 0; c < CT; ++c) w[ks][c] = *reinterpret_cast<const bf16x8_t*>(stage + (ks ? rw ^ 64u : rw) + c * 2048);
#pragma unroll
                    for (int i = 0; i < RT; ++i) x[ks][i] = *reinterpret_cast<const bf16x8_t*>(lds + (ks ? r1 : r0) + i * (16 * PITCH));
                }
                r0 += 128u; r1 += 128u;
                __builtin_amdgcn_sched_barrier(0);
            };
            // the stage's operands are in registers: its place is refilled, the next stage's are requested, then the products
            auto stage = [&](const bf16x8_t (&x)[2][RT], const bf16x8_t (&w)[2][CT], bf16x8_t (&xn)[2][RT], bf16x8_t (&wn)[2][CT], bool more) {
                __builtin_amdgcn_s_waitcnt(0xc07f);       // lgkmcnt(0), in a form that the compiler counts too
                __builtin_amdgcn_sched_barrier(0);
                if (pos == kn) { set_unit(t + step); pos = 0; }
                load(slot); ++pos;
                slot = slot == ND - 1 ? 0 : slot + 1;
                __builtin_amdgcn_sched_barrier(0);
                if (more) read(xn, wn);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int c = 0; c < CT; ++c)
#pragma unroll
                        for (int i = 0; i < RT; ++i)
                            acc[i][c] = TOKENS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[ks][i], w[ks][c], acc[i][c], 0, 0, 0)
                                               : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][c], x[ks][i], acc[i][c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            if (kn > 0) read(fa[0], fb[0]);
#pragma unroll 1
            for (int k = 0; k < kn; k += 2) {
                stage(fa[0], fb[0], fa[1], fb[1], k + 1 < kn);
                if (k + 1 < kn) stage(fa[1], fb[1], fa[0], fb[0], k + 2 < kn);
            }
        };
        // positions and addresses of the rows are worked out per column tile, not kept in registers over the products
        int e16 = l16, eq = lq;
        auto place = [&]() { asm volatile("" : "+v"(e16), "+v"(eq)::"memory"); };
        bf16_t* const out = sect == 0 ? a.out[0] : sect == 1 ? a.out[1] : a.out[2];
        const int scol = col - sect * a.sect_n;
        run();
        if (g.ks) {                                       // the parts' sums meet in the place of the rows; the first part's wave goes on
            f32x4_t* const sums = reinterpret_cast<f32x4_t*>(lds);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (part)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int c = 0; c < CT; ++c) sums[(wave * (RT * CT) + i * CT + c) * 64 + lane] = acc[i][c];
            __syncthreads();
            if (part) { t = t1; return; }
            for (int o = 1; o < 1 << g.ks; ++o)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int c = 0; c < CT; ++c) acc[i][c] += sums[((wave + o) * (RT * CT) + i * CT + c) * 64 + lane];
        }
        place();
        u32x2_t bias[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            bias[c] = u32x2_t{0, 0};
            if constexpr (BIAS) bias[c] = *reinterpret_cast<const u32x2_t*>(lbias + ((t - t0) * OC + eq * 4 + (c == 0 ? 0 : GEGLU ? g.per * OC : c * 16)) * 2);
        }
        if constexpr (GEGLU) {
            const float bv[4] = {lo16(bias[0].x), hi16(bias[0].x), lo16(bias[0].y), hi16(bias[0].y)};
            const float bg[4] = {lo16(bias[1].x), hi16(bias[1].x), lo16(bias[1].y), hi16(bias[1].y)};
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int gm = m0 + i * 16 + e16;
                float y[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) y[q] = (acc[i][0][q] + bv[q]) * gelu_f(acc[i][CT - 1][q] + bg[q]);
                if (gm < rows) *(FISE_AS1 u32x2_t*)(out + (size_t)gm * a.N + col + eq * 4) = u32x2_t{f2bf2(y[0], y[1]), f2bf2(y[2], y[3])};
            }
        } else if constexpr (TOKENS) {
            const size_t HW = (size_t)a.Ho * a.Wo;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int r = i * 16 + eq * 4;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const unsigned n = (unsigned)(scol + c * 16 + e16);
                    if (g.trans4) {                       // four tokens in a row
                        const int2 pos = rowpos[r];
                        if (m0 + r < rows)
                            *(FISE_AS1 u32x2_t*)(out + ((size_t)pos.x * a.sect_n + n) * HW + pos.y) = u32x2_t{f2bf2(acc[i][c][0], acc[i][c][1]), f2bf2(acc[i][c][2], acc[i][c][3])};
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int2 pos = rowpos[r + q];
                            if (m0 + r + q < rows) *(FISE_AS1 bf16_t*)(out + ((size_t)pos.x * a.sect_n + n) * HW + pos.y) = f2bf(acc[i][c][q]);
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int r = i * 16 + e16;
                const int2 pos = rowpos[r];
                const size_t row = mode == OUT_MAP ? (size_t)pos.x * (a.Ho * a.Wo) + pos.y : (size_t)(m0 + r);
                if (m0 + r >= rows) continue;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const f32x4_t y = acc[i][c] + f32x4_t{lo16(bias[c].x), hi16(bias[c].x), lo16(bias[c].y), hi16(bias[c].y)};
                    const size_t off = row * a.sect_n + scol + c * 16 + eq * 4;
                    if (mode == OUT_COMPACT_F32) *(FISE_AS1 f32x4_t*)(reinterpret_cast<float*>(out) + off) = y;
                    else *(FISE_AS1 u32x2_t*)(out + off) = u32x2_t{f2bf2(y[0], y[1]), f2bf2(y[2], y[3])};
                }
            }
        }
        t += step;
    };
    // the transposed section is the last one: two loops instead of a choice in one, which costs copies of the ring
    const bool idle = t >= t1;
    while (t < min(t1, g.t_tokens)) column_tile(std::false_type{});
    if constexpr (!GEGLU)
        while (t < t1) column_tile(std::true_type{});
    if (g.ks && idle) {                                   // every wave meets the two barriers of a split unit
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        __syncthreads();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the loads past the range still write to this workgroup's LDS
#endif
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int KM, int RT, int CT, int ND> constexpr int ng_lds(bool bias, bool table) {
    return 16 * RT * (ng_pitch<KM>() + 8) + NG_WAVES * ND * CT * 2048 + (bias ? NG_BIAS : 0) + (table ? 2 * 320 * KM * 8 : 0);
}

template <int KM, int RT, int CT, int ND, bool GEGLU, int SRC>
static int launch_cfg(NormGemmDev g, int per, hipStream_t st) {
    const NormGemmArgs& a = g.a;
    constexpr int lds = ng_lds<KM, RT, CT, ND>(norm_gemm_has_bias(GEGLU, SRC), SRC == NG_MAP_GN);
    static_assert(SRC == NG_MAP_GN || lds <= NG_LDS_MAX, "LDS of a CU");
    if constexpr (lds > NG_LDS_MAX) {                    // a table that finds no room: choose_norm_tile passes the tile by
        return fail(FISE_ERR_SHAPE, "norm gemm: LDS of a CU");
    } else {
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&norm_gemm_kernel<KM, RT, CT, ND, GEGLU, SRC>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (attr != hipSuccess) return fail(FISE_ERR_HIP, "norm gemm: cannot raise the dynamic LDS limit");
        const int rows = a.B * a.Ma;
        g.gx = ceil_div(rows, 16 * RT); g.units = a.N / (GEGLU ? 16 : 16 * CT); g.per = per;
        g.t_tokens = a.mode[a.N / a.sect_n - 1] == OUT_TOKENS_T ? (a.N - a.sect_n) / (16 * CT) : g.units;
        g.touch = g.gx >= 3 && per * CT * KM * 10 >= 200;      // kernel comment
        g.ks = waves_per_unit(KM, CT, per);
        g.d_gx = fast_div(g.gx);
        {
            const double K = 320.0 * KM, ncols = GEGLU ? 2.0 * a.N : a.N;
            ProfileScope prof(GEGLU ? PROF_IGEMM_GEGLU : PROF_ROWS_GEMM, 2.0 * rows * ncols * K,
                              2.0 * (ncols * K + (double)rows * a.N) + (SRC == NG_ROWS_LN ? 4.0 : 2.0) * rows * K, st);
            hipLaunchKernelGGL((norm_gemm_kernel<KM, RT, CT, ND, GEGLU, SRC>), dim3((unsigned)(g.gx * ceil_div(g.units, per))), dim3(64 * NG_WAVES), lds, st, g);
        }
        FISE_CHECK_LAUNCH("norm gemm");
        return FISE_OK;
    }
}

// the gate rides on the LayerNorm of the residual stream only
template <int KM, int RT, int CT, int ND, bool GEGLU>
static int launch_src(const NormGemmDev& g, int per, hipStream_t st) {
    if constexpr (!GEGLU) {
        if (g.a.src == NG_MAP_LN) return launch_cfg<KM, RT, CT, ND, false, NG_MAP_LN>(g, per, st);
        if (g.a.src == NG_MAP_GN) return launch_cfg<KM, RT, CT, ND, false, NG_MAP_GN>(g, per, st);
        if (g.a.src == NG_MAP_RAW) return launch_cfg<KM, RT, CT, ND, false, NG_MAP_RAW>(g, per, st);
    }
    return launch_cfg<KM, RT, CT, ND, GEGLU, NG_ROWS_LN>(g, per, st);
}

#define FISE_NORM_LAUNCH(K, GEGLU, RT, CT, ND) launch_src<K / 320, RT, CT, ND, GEGLU != 0>,
static int (*const kNormLaunch[])(const NormGemmDev&, int, hipStream_t) = {FISE_NORM_TILES(FISE_NORM_LAUNCH)};
#undef FISE_NORM_LAUNCH

bool norm_gemm_takes(int src, int K, int B, int Ma, int H, int W) {
    if ((K != 320 && K != 640 && K != 1280) || Ma < 1) return false;
    if (src == NG_MAP_GN && B > 1 && Ma < (K == 1280 ? 16 : 32)) return false;
    return (long long)B * Ma < 1 << 24 && (long long)B * H * W < 1 << 24;       // 32-bit products of row and pixel numbers
}

int launch_norm_gemm(const NormGemmArgs& a, hipStream_t st) {
    NormGemmDev g{};
    g.a = a;
    const int nsect = a.N / a.sect_n;
    bool map = a.src != NG_ROWS_LN, tokens = false;
    for (int s = 0; s < nsect; ++s) { map |= a.mode[s] == OUT_MAP; tokens |= a.mode[s] == OUT_TOKENS_T; if (a.mode[s] == OUT_TOKENS_T && s + 1 < nsect) return fail(FISE_ERR_SHAPE, "norm gemm: a transposed section is the last one"); }
    if (!norm_gemm_takes(a.src, a.K, a.B, a.Ma, a.Ho, a.Wo) || a.sect_n % 32 || nsect * a.sect_n != a.N || nsect > 3 || (a.geglu && (nsect != 1 || a.src != NG_ROWS_LN)) || (a.bias && nsect != 1))
        return fail(FISE_ERR_SHAPE, "norm gemm: %d channels, %d columns in sections of %d", a.K, a.N, a.sect_n);
    if (a.bias && !norm_gemm_has_bias(a.geglu != 0, a.src)) return fail(FISE_ERR_SHAPE, "norm gemm: a bias behind a LayerNorm without a gate");
    g.pixels = a.tile_idx && (map || tokens);
    g.trans4 = a.Ma % 4 == 0 && (a.tile_idx ? a.tile % 4 == 0 && a.Wo % 4 == 0 : a.Ho * a.Wo % 4 == 0);
    g.d_Ma = fast_div(a.Ma); g.d_tt = fast_div(a.tile * a.tile); g.d_tile = fast_div(a.tile); g.d_tiles_w = fast_div(a.tiles_w);
    g.d_cpg = fast_div(a.src == NG_MAP_GN ? a.K / a.G : 1);
    const NormChoice c = choose_norm_tile({a.B, a.Ma, a.K, a.N, a.geglu != 0, a.src == NG_MAP_GN});
    if (c.tile < 0) return fail(FISE_ERR_SHAPE, "norm gemm: no tile");
    return kNormLaunch[c.tile](g, c.per, st);
}

}  // namespace fise
