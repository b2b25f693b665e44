// 3x3 convolutions (stride 1, square tiles of edge 4 or 8) of many rows, output widths that are multiples of 80: tiles of 64 or 128 rows x
// 80 columns.  As in the patch form of wave_gemm.hip a tile's pixels and their ring come into LDS once per 64 channels and are read under
// all nine taps; the weights of a tap (80 rows of 128 bytes) run through a ring of their own, a tap at a time.
// What a CU gets through LDS-direct loads (71 - 88 GB/s) bounds every form of these convolutions, so the bytes per product decide: 128 x 80
// outputs bring in 13 KB a tap (10 of weights, 3 of pixels), 64 x 160 gathered 28 KB; and 80 columns divide widths of 320, 640 and 1280
// without a remainder, so 8192 x 320 and 2048 x 640 outputs are one tile for each of the 256 CUs.
//  - Four waves: two share K (32 of the 64 channels each), two the rows; 16 x 16 x 32 products, a wave's operands of the next tap are read
//    from LDS while the matrix pipe works on this one.
//  - A 1x1 side product (the block's shortcut) follows as a plain product over the same LDS.
//  - The two K halves of a row meet in LDS, each finishing half of the row tiles.
#include <type_traits>
#include "igemm.h"
#include "patch.h"
#include "profile.h"

namespace fise {

constexpr int CP_TAP = 80 * 128, CP_STEP = 3 * CP_TAP;       // bytes of a tap's weights, of a kernel row's
[[maybe_unused]] constexpr int CP_LW = 8;   // loads of a kernel row's weights per wave: 30 of 1 KB, dealt out (two are loads of nothing)
template <int RT, int T> struct ConvPatch {
    static constexpr int BM = 32 * RT, SIDE = (BM + 80) * 128, RING = 2 * Patch<BM, T>::BYTES + 3 * CP_STEP, NS = RING / SIDE < 4 ? RING / SIDE : 4;
    static constexpr int LDS = RING + 1024 + BM * 8;    // patches, weights, a place for loads of nothing, the rows' positions
    // Segment of 16 bytes that slot 0 of patch row p holds: the sixteen lanes that the LDS serves at once (sixteen pixels, eight of them of one
    // segment, eight of the next) meet in no bank under any tap.
    static __device__ __forceinline__ int swizzle(int p) {
        const int q = p % Patch<BM, T>::PIX;
        return (q % (T + 2) / 2 * 2 + (T == 4 ? 4 * (q / (T + 2)) : 0)) & 7;
    }
};
template <int RT, int T>
__global__ __launch_bounds__(256, 1) void conv_patch_kernel(const IgemmArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using G = ConvPatch<RT, T>;
    constexpr int BM = G::BM, CT = 5, NS = G::NS;
    using PG = Patch<BM, T>;
    constexpr unsigned OOB = 0x80000000u;
    static_assert(PG::H == T && NS >= 3, "whole tiles");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    unsigned char* const wring = lds + 2 * PG::BYTES;
    unsigned char* const nowhere = lds + G::RING;
    int2* const rowpos = reinterpret_cast<int2*>(lds + G::RING + 1024);
    asm volatile("" ::"s"(a.gx), "s"(a.gy), "s"(a.d_gx.mul), "s"(a.d_Ma.mul), "s"(a.d_tt.mul), "s"(a.d_tiles_w.mul), "s"(a.B), "s"(a.Ma), "s"(a.K), "s"(a.K2),
                 "s"(a.N), "s"(a.w), "s"(a.tile_idx), "s"(a.Ho), "s"(a.Wo), "s"(a.C0), "s"(a.C1), "s"(a.touch));
    asm volatile("" ::"s"(a.bias), "s"(a.bias_bytes), "s"(a.bias2), "s"(a.bias2_bytes), "s"(a.temb), "s"(a.temb_bytes), "s"(a.res), "s"(a.res_bytes), "s"(a.nview),
                 "s"(a.src[0].p), "s"(a.src[0].bytes), "s"(a.src[0].pitch), "s"(a.out[0]));
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4, l8 = lane >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kh = wave & 1, mw = wave >> 1;
    const int total = a.gx * a.gy, run = total >> 3;     // every XCD gets a contiguous run of (columns, rows), rows fastest
    int w = blockIdx.x;
    if (w < (run << 3)) w = (w & 7) * run + (w >> 3);
    const int by = (int)fdiv((unsigned)w, a.d_gx), bx = w - by * a.gx;
    const int rows = a.B * a.Ma, m0 = bx * BM, nchunk = a.K / 576;

    // ---- patches: every lane's rows (tile, pixel in the ringed tile); all tile numbers are requested together
    int tile_no[PG::SLOTS];
#pragma unroll
    for (int j = 0; j < PG::SLOTS; ++j) {
        const int p = j * 32 + wave * 8 + l8;
        const unsigned m = (unsigned)min(m0 + p / PG::PIX * (T * T), rows - 1), b = fdiv(m, a.d_Ma);
        tile_no[j] = ((const FISE_AS1 int*)a.tile_idx)[fdiv(m - b * (unsigned)a.Ma, a.d_tt)];
    }
    const unsigned row = (unsigned)min(m0 + min(tid, BM - 1), rows - 1), row_b = fdiv(row, a.d_Ma), row_m = row - row_b * (unsigned)a.Ma, row_t = fdiv(row_m, a.d_tt);
    const unsigned row_no = (unsigned)((const FISE_AS1 int*)a.tile_idx)[row_t];
    // ---- weights: a step is the three taps of a kernel row, 30 pieces of eight rows; wave w loads the pieces w, w + 4 ...
    const unsigned pitch_w = (unsigned)a.K * 2u, tap_bytes = (unsigned)(a.C0 + a.C1) * 2u;
    unsigned vb[CP_LW];
#pragma unroll
    for (int l = 0; l < CP_LW; ++l) {
        const int g = wave + 4 * l, r = g % 10 * 8 + l8;
        vb[l] = g < 30 ? __umul24((unsigned)(by * 80 + r), pitch_w) + (unsigned)(g / 10) * tap_bytes + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16) : OOB;
    }
    const unsigned wbytes = __umul24((unsigned)a.N, pitch_w);
    auto issue_w = [&](int chunk, int ky) {              // into slot ky; chunks past the last: a descriptor of size zero, no traffic
        const __amdgpu_buffer_rsrc_t rs = buf(a.w, chunk < nchunk ? wbytes : 0u);
        const unsigned soff = (unsigned)chunk * 128u + (unsigned)ky * 3u * tap_bytes;
#pragma unroll
        for (int l = 0; l < CP_LW; ++l)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(l < 7 || wave < 2 ? wring + ky * CP_STEP + (wave + 4 * l) * 1024 : nowhere), 16, vb[l], soff, 0, 0);
    };
    // the row tiles of a column first touch its weights, each a share of the lines (as in wave_gemm.hip)
    if (a.touch) {
        const __amdgpu_buffer_rsrc_t rs = buf(a.w, wbytes);
        const int lines = a.K >> 6;                      // of 128 bytes in a row
        for (int q = (bx * 4 + wave) * 64 + lane; q < 80 * lines; q += a.gx * 256) {
            const int r = q / lines;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)nowhere, 4, __umul24((unsigned)(by * 80 + r), pitch_w) + (unsigned)(q - r * lines) * 128u, 0, 0, 0);
        }
    }
    issue_w(0, 0);

    unsigned px[PG::SLOTS], va[PG::SLOTS], soff_p = 0, end_p = 0; const bf16_t* ptr_p = nullptr; unsigned bytes_p = 0; int chunk_p = 0;
#pragma unroll
    for (int j = 0; j < PG::SLOTS; ++j) {
        const int p = j * 32 + wave * 8 + l8, strip = p / PG::PIX, q = p - strip * PG::PIX, m = m0 + strip * (T * T);
        const unsigned b = fdiv((unsigned)min(m, rows - 1), a.d_Ma), ty = fdiv((unsigned)tile_no[j], a.d_tiles_w);
        const int iy = (int)ty * T - 1 + q / (T + 2), ix = (tile_no[j] - (int)ty * a.tiles_w) * T - 1 + q % (T + 2);
        const bool in = strip < PG::STRIPS && m < rows && (unsigned)iy < (unsigned)a.Ho && (unsigned)ix < (unsigned)a.Wo;
        px[j] = in ? (b * (unsigned)a.Ho + iy) * (unsigned)a.Wo + ix | (unsigned)((lane & 7) ^ G::swizzle(p)) << 24 : OOB;
    }
    if (tid < BM) {                                      // the rows' positions, for the side product and the epilogue
        const unsigned rp = row_m - row_t * (T * T), ty = fdiv(row_no, a.d_tiles_w);
        const unsigned pix = (row_b * (unsigned)a.Ho + ty * T + rp / T) * (unsigned)a.Wo + (row_no - ty * a.tiles_w) * T + rp % T;
        rowpos[tid] = make_int2((int)row_b, m0 + tid < rows ? (int)pix : -1);
    }
    auto set_source = [&](int i) {
        ptr_p = a.src[i].p; bytes_p = a.src[i].bytes; end_p = a.src[i].pitch; soff_p = 0;
#pragma unroll
        for (int j = 0; j < PG::SLOTS; ++j) va[j] = (__umul24(px[j], end_p) + (px[j] >> 20 & 0x70u)) | (px[j] & OOB);
    };
    auto issue_patch = [&]() {
        const __amdgpu_buffer_rsrc_t rs = buf(ptr_p, chunk_p < nchunk ? bytes_p : 0u);
        unsigned char* const base = lds + (chunk_p & 1) * PG::BYTES + wave * 1024;
#pragma unroll
        for (int j = 0; j < PG::SLOTS; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + j * 4096), 16, va[j], soff_p, 0, 0);
        ++chunk_p; soff_p += 128u;
        if (soff_p == end_p && chunk_p < nchunk) set_source(1);
    };
    set_source(0);
    issue_patch();
    issue_w(0, 1);
    issue_w(0, 2);
    issue_patch();
    __builtin_amdgcn_sched_barrier(0);

    // ---- K loop
    f32x4_t acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[i][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    unsigned rp[9][RT];                                  // operand A under each tap: place in a patch
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int r = (mw * RT + i) * 16 + l16, q = r / (T * T) * PG::PIX + r % (T * T) / T * (T + 2) + r % T;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int p = q + t / 3 * (T + 2) + t % 3;
            rp[t][i] = (unsigned)(p * 128 + (((kh * 4 + lq) ^ G::swizzle(p)) * 16));
        }
    }
    const unsigned rw = (unsigned)(l16 * 128 + (((kh * 4 + lq) ^ ((l16 >> 1) & 7)) * 16));      // operand W within 16 rows
    bf16x8_t fa[2][RT], fb[2][CT];
    unsigned rpatch = 0;                                 // patch whose operands are read next
    auto multiply = [&](const bf16x8_t (&x)[RT], const bf16x8_t (&y)[CT], int c) {
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[c], x[i], acc[i][c], 0, 0, 0);
    };
    // W and A of a tap in turn
    constexpr int OPS = CT + RT;
    auto operand = [&](bf16x8_t (&x)[RT], bf16x8_t (&y)[CT], int tap, int k) {
        if (k < 2 * RT && (k & 1)) x[k >> 1] = *reinterpret_cast<const bf16x8_t*>(lds + rpatch + rp[tap][k >> 1]);
        else { const int c = k < 2 * RT ? k >> 1 : k - RT; y[c] = *reinterpret_cast<const bf16x8_t*>(wring + tap * CP_TAP + rw + c * 2048); }
    };
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * CP_LW + PG::SLOTS) : "memory");      // all but the second and third step's weights and the second patch
#pragma unroll
    for (int k = 0; k < OPS; ++k) operand(fa[0], fb[0], 0, k);
    // A chunk whose first operands lie in register set P.  In the third tap of a kernel row every wave has that row's operands in registers: behind
    // a barrier there its place in the ring takes the same row of the next chunk, behind the last row's the patch that of the chunk after next.  The
    // wait in front of that barrier is for the next row, requested six taps ago (and a patch nine): only what was requested since may be in flight.
    auto chunk = [&](auto first, int c) {
        constexpr int P = decltype(first)::value;
        auto step = [&](auto tap) {
            constexpr int s = decltype(tap)::value, cur = (P + s) & 1, ky = s / 3, nt = s == 8 ? 0 : s + 1, PER = (OPS + 2) / 3;
            __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0): this tap's operands
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (s % 3 == 2) {
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(ky == 2 ? CP_LW : CP_LW + PG::SLOTS) : "memory");
                if (s == 8) rpatch ^= (unsigned)PG::BYTES;
            }
            // The next operands are requested between the products, a few at a time: in one go the wave would stand at the LDS until they
            // are served before its first product.  Behind the last tap: not used.
#pragma unroll
            for (int n = 0; n < CT; ++n) {
                multiply(fa[cur], fb[cur], n);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = n * PER; k < (n + 1) * PER && k < OPS; ++k) operand(fa[cur ^ 1], fb[cur ^ 1], nt, k);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (s % 3 == 2) {
                    if (n == 1) issue_w(c + 1, ky);
                    if (n == 3 && s == 8) issue_patch();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{}); step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{}); step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
        step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 7>{}); step(std::integral_constant<int, 8>{});
    };
#pragma unroll 1
    for (int c = 0; c < nchunk; c += 2) {
        chunk(std::integral_constant<int, 0>{}, c);
        if (c + 1 < nchunk) chunk(std::integral_constant<int, 1>{}, c + 1);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- side product: stages of BM rows of the raw maps at the output pixels and 80 rows of w2, 64 channels each
    if (a.K2 > 0) {
        const unsigned pitch2 = (unsigned)a.K2 * 2u, w2bytes = __umul24((unsigned)a.N, pitch2);
        unsigned pix[RT], vs[RT], v2[3];
#pragma unroll
        for (int l = 0; l < RT; ++l) pix[l] = (unsigned)rowpos[(wave + 4 * l) * 8 + l8].y;      // -1: no such row
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const int g = wave + 4 * l, r = g * 8 + l8;
            v2[l] = g < 10 ? __umul24((unsigned)(by * 80 + r), pitch2) + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16) : OOB;
        }
        const int nside = a.K2 >> 6;
        int issued = 0; unsigned soff = 0, slot = 0, end = 0; const bf16_t* ptr = nullptr; unsigned bytes = 0;
        auto source = [&](int i) {
            ptr = a.src[i].p; bytes = a.src[i].bytes; end = a.src[i].pitch; soff = 0;
#pragma unroll
            for (int l = 0; l < RT; ++l) {
                const int r = (wave + 4 * l) * 8 + l8;
                vs[l] = (int)pix[l] < 0 ? OOB : __umul24(pix[l], end) + (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
            }
        };
        auto issue = [&]() {
            const bool live = issued < nside;
            const __amdgpu_buffer_rsrc_t rs = buf(ptr, live ? bytes : 0u), r2 = buf(a.w2, live ? w2bytes : 0u);
            unsigned char* const base = lds + slot;
#pragma unroll
            for (int l = 0; l < RT; ++l) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + (wave + 4 * l) * 1024), 16, vs[l], soff, 0, 0);
#pragma unroll
            for (int l = 0; l < 3; ++l)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r2, (__attribute__((address_space(3))) void*)(wave + 4 * l < 10 ? base + BM * 128 + (wave + 4 * l) * 1024 : nowhere), 16, v2[l], (unsigned)issued * 128u, 0, 0);
            ++issued; soff += 128u;
            if (soff == end && issued < nside) source(3);
            slot = slot == (NS - 1) * G::SIDE ? 0u : slot + G::SIDE;
        };
        source(2);
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue();
        unsigned rs = 0;
#pragma unroll 1
        for (int k = 0; k < nside; ++k) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * (RT + 3)) : "memory");
#pragma unroll
            for (int c = 0; c < CT; ++c) fb[0][c] = *reinterpret_cast<const bf16x8_t*>(lds + rs + BM * 128 + rw + c * 2048);
#pragma unroll
            for (int i = 0; i < RT; ++i) fa[0][i] = *reinterpret_cast<const bf16x8_t*>(lds + rs + (mw * RT + i) * 2048 + rw);
            rs = rs == (NS - 1) * G::SIDE ? 0u : rs + G::SIDE;
            __builtin_amdgcn_sched_barrier(0);
            issue();                                     // the place of stage k - 1, which every wave has in registers
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < CT; ++c) multiply(fa[0], fb[0], c);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }

    // ---- the K halves: each wave finishes RT / 2 of its row tiles and hands over the others
    constexpr int HT = RT / 2;
    f32x4_t* const hand = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) hand[((wave * HT + i) * CT + c) * 64 + lane] = kh ? acc[i][c] : acc[HT + i][c];
    __syncthreads();
    u32x2_t e_bias[CT], e_bias2[CT];
    {
        const __amdgpu_buffer_rsrc_t s1 = buf(a.bias, a.bias_bytes), s2 = buf(a.bias2, a.bias2_bytes);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const unsigned col = (unsigned)(by * 80 + c * 16 + lq * 4);
            e_bias[c] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s1, col * 2u, 0, 0));
            e_bias2[c] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s2, col * 2u, 0, 0));
        }
    }
    const __amdgpu_buffer_rsrc_t s_temb = buf(a.temb, a.temb_bytes), s_res = buf(a.res, a.res_bytes);
#pragma unroll
    for (int i = 0; i < HT; ++i) {
        const int2 pos = rowpos[(mw * RT + kh * HT + i) * 16 + l16];
        const unsigned no = pos.y < 0 ? OOB : 0u, pix = (unsigned)max(pos.y, 0);
        u32x2_t e_res[CT]; f32x4_t e_temb[CT]; u32x4_t ss[2][CT][2];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const unsigned col = (unsigned)(by * 80 + c * 16 + lq * 4);
            e_res[c] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s_res, ((__umul24(pix, (unsigned)a.N) + col) * 2u) | no, 0, 0));
            e_temb[c] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s_temb, (__umul24((unsigned)pos.x, (unsigned)a.temb_stride) + col) * 4u, 0, 0));
        }
#pragma unroll
        for (int v = 0; v < 2; ++v)
            if (v < a.nview) {
                const __amdgpu_buffer_rsrc_t s = buf(a.view[v].ss, (unsigned)a.B * a.view[v].dstC * 8u);
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const unsigned off = (__umul24((unsigned)pos.x, (unsigned)a.view[v].dstC) + a.view[v].c_off + by * 80 + c * 16 + lq * 4) * 8u;
                    ss[v][c][0] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s, off, 0, 0));
                    ss[v][c][1] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s, off, 16, 0));
                }
            }
        u32x2_t y[CT], u[2][CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const f32x4_t own = kh ? acc[HT + i][c] : acc[i][c], sum = own + hand[(((wave ^ 1) * HT + i) * CT + c) * 64 + lane];
            float x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                auto part = [q](const u32x2_t& v) { return q & 1 ? hi16(v[q >> 1]) : lo16(v[q >> 1]); };
                x[q] = sum[q] + part(e_bias[c]);
                x[q] += part(e_bias2[c]);
                x[q] += part(e_res[c]) + e_temb[c][q];
            }
            y[c] = u32x2_t{f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
#pragma unroll
            for (int v = 0; v < 2; ++v)
                if (v < a.nview) {                       // as put_views4
                    float z[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        z[q] = view_scale(q & 1 ? hi16(y[c][q >> 1]) : lo16(y[c][q >> 1]), __uint_as_float(ss[v][c][q >> 1][(q & 1) * 2]), __uint_as_float(ss[v][c][q >> 1][(q & 1) * 2 + 1]));
                    if (a.view[v].silu)
#pragma unroll
                        for (int q = 0; q < 4; ++q) z[q] = silu_f(z[q]);
                    u[v][c] = u32x2_t{f2bf2(z[0], z[1]), f2bf2(z[2], z[3])};
                }
        }
        if (pos.y >= 0)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const unsigned col = (unsigned)(by * 80 + c * 16 + lq * 4);
                *(FISE_AS1 u32x2_t*)(a.out[0] + (size_t)pix * a.N + col) = y[c];
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    if (v < a.nview) *(FISE_AS1 u32x2_t*)(a.view[v].dst + (size_t)pix * a.view[v].dstC + a.view[v].c_off + col) = u[v][c];
            }
    }
#endif
}

template <int RT, int T>
static int launch_cp(const IgemmArgs& a, hipStream_t st) {
    constexpr int lds = ConvPatch<RT, T>::LDS;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_patch_kernel<RT, T>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "conv patch: cannot raise the dynamic LDS limit");
    const double rows = (double)a.B * a.Ma, K = (double)a.K + a.K2;
    {
        ProfileScope prof(PROF_IGEMM, 2.0 * rows * a.N * K, 2.0 * (a.N * K + rows * (a.C0 + a.C1 + a.S0 + a.S1) + rows * a.N), st);
        hipLaunchKernelGGL((conv_patch_kernel<RT, T>), dim3((unsigned)(a.gx * a.gy)), dim3(256), lds, st, a);
    }
    FISE_CHECK_LAUNCH("conv patch");
    return FISE_OK;
}

int launch_conv_patch(const IgemmArgs& a, int tm, hipStream_t st) {
    if (tm == 4) return launch_cp<4, 8>(a, st);
    return a.tile == 8 ? launch_cp<2, 8>(a, st) : launch_cp<2, 4>(a, st);
}

}  // namespace fise
