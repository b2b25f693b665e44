// Gathered GEMM for tiles of 32 or 64 rows whose K loop is split over the waves of ONE workgroup.
//
//   out[row, n] = epilogue( sum_k A[row, k] * W[n, k]  (+ sum_k A2[row, k] * W2[n, k]) )      (see igemm.h)
//
// What bounds the masked step is not bandwidth or MFMA rate but the fixed cost of 277 dependent launches (178 of them this
// kernel), and inside a launch the round trips to memory.  So this kernel is built around them.  What a CU gets through LDS-direct
// loads depends on who else is at it (operand bytes over time, tiles of 32 x 32 to 64 x 160): 71 - 88 GB/s over a launch with all
// 256 CUs busy (18 - 22 TB/s together), 110 in the K loop of 240 workgroups whose lines are in L2 (85 where they are not), 125
// alone out of its L2.
//  - Every wave owns the whole 32*TM x 32*TN tile for its share of K and runs it from an LDS ring of its own, filled by
//    LDS-direct loads: no barrier in the K loop, a wave waits for its own loads only, and 4 waves x 2 stages of 8 - 16 KB keep
//    32 - 128 KB per CU in flight (32 KB are enough for the 125 GB/s of a CU alone).
//  - No row table and no barrier in front of the first load: the lanes work out their own rows (divisions by
//    precomputed reciprocals), the weight loads of the first stages go out before the pixel of a row is known.
//  - Everything the epilogue fetches (biases, time projection, residual, scale / shift tables) is requested before the K
//    loop through buffer descriptors; an operand that is absent has a descriptor of size zero, so there is no branch and
//    hence no round trip per operand.
//  - The waves' partial tiles are summed through LDS in wave order.  Where the tiles of a launch do not fill the chip K is
//    also split over workgroups: every workgroup parks its tile (written through to memory), counts itself on a per-tile
//    counter, and the one that arrives last adds the parked tiles in split order and finishes.  Nobody waits for anybody,
//    so there is nothing to deadlock, and the sum does not depend on who came last.
// Measured against shared 64x64 tiles with a reduce launch behind every K split: step of 12 of 64 tiles 3070 -> 2590 us,
// 2 of 70 tiles 2600 -> 1985 us, transformer block of 160 rows 92 -> 78 us.
#include <algorithm>
#include "igemm.h"
#include "profile.h"

namespace fise {

#define FISE_AS1 __attribute__((address_space(1)))
typedef unsigned u32x2_w __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_w __attribute__((ext_vector_type(4)));
typedef float f32x4_w __attribute__((ext_vector_type(4)));

enum { A_ROWS = 0, A_MAP = 1 };         // compact rows / pixels of maps (taps, two sources, side product)

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float lo16(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ float gelu_f(float x) { return x * (0.5f * (1.0f + erff(x * 0.70710678118654752f))); }
#endif

// SHARED: one ring for the workgroup instead of one per wave, see the launcher.
template <int TM, int TN, int NW, int NST, int AM, bool GEGLU, bool SHARED>
__global__ __launch_bounds__(64 * NW, SHARED && TN == 2 ? 3 : 1) void wave_gemm_kernel(const IgemmArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 32 * TM, BN = 32 * TN, NT = 64 * NW;
    constexpr int RB = SHARED ? 8 * NW : 8;             // rows between two loads of a lane (one load of a wave fills 8 rows of 128 bytes)
    constexpr int AL = BM / RB, BL = BN / RB;           // 16-byte loads per lane and K step
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int PITCH = BN + 4;                       // floats per row of a partial tile in LDS
    constexpr int OW = GEGLU ? BN / 2 : BN;             // output columns of the tile
    constexpr int GROUPS = SHARED ? TM : 1, GROWS = BM / GROUPS;       // the waves' sums are finished in groups of rows: what fits in the ring
    constexpr int CPR = OW / 4, IPG = GROWS * CPR / NT, ITEMS = GROUPS * IPG;      // four-column pieces per row, per thread and group, per thread
    constexpr unsigned OOB = 0x80000000u;               // beyond every descriptor: the load returns zeros
    static_assert(GROWS * CPR % NT == 0 && (SHARED ? 1 : NW) * NST * STAGE >= NW * GROWS * PITCH * 4, "tile");
    constexpr bool CONV = TN == 5;                      // the block tile: one map out, bf16 map as residual
    static_assert(!SHARED || (NW == 4 && NST >= 3), "a shared stage has one 16-deep slice of K per wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];      // [NW or 1][NST][STAGE], later [NW][GROWS][PITCH] floats

    // Kernel arguments arrive through scalar loads placed where a field is first used; named here they come as one batch.
    asm volatile("" ::"s"(a.gx), "s"(a.gy), "s"(a.splits), "s"(a.kper), "s"(a.d_gx.mul), "s"(a.d_gy.mul), "s"(a.d_Ma.mul), "s"(a.d_tt.mul),
                 "s"(a.d_tw.mul), "s"(a.d_tiles_w.mul), "s"(a.B), "s"(a.Ma), "s"(a.K), "s"(a.K2), "s"(a.N), "s"(a.w), "s"(a.tile_idx), "s"(a.need_pix));
    asm volatile("" ::"s"(a.Ho), "s"(a.Wo), "s"(a.tile), "s"(a.sect_n), "s"(a.out_mode[0]), "s"(a.bias), "s"(a.bias_bytes), "s"(a.temb), "s"(a.temb_bytes),
                 "s"(a.res), "s"(a.res_bytes), "s"(a.res_compact), "s"(a.nview), "s"(a.src[0].p), "s"(a.src[0].bytes));
    if constexpr (AM == A_MAP) asm volatile("" ::"s"(a.Hin), "s"(a.Win), "s"(a.ksize), "s"(a.stride), "s"(a.ups), "s"(a.C0), "s"(a.d_spt.mul), "s"(a.bias2), "s"(a.bias2_bytes));
    const int tid = threadIdx.x, lane = tid & 63, lr = lane >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive workgroups go round-robin to the 8 XCDs: give every XCD a contiguous run of (bz, by, bx), bx fastest, so
    // that a slice of the weights is pulled into one L2
    int bx, by, bz;
    {
        const int total = a.gx * a.gy * a.splits, chunk = total >> 3;
        int w = blockIdx.x;
        if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
        const unsigned t = fdiv((unsigned)w, a.d_gx);
        bx = w - (int)t * a.gx; bz = (int)fdiv(t, a.d_gy); by = (int)t - bz * a.gy;
    }
    const int rows = a.B * a.Ma, m0 = bx * BM;
    const int nsteps1 = a.K >> 6, nsteps = nsteps1 + (a.K2 >> 6);
    int kb, ke;                                         // K steps of this wave
    {
        const int c0 = bz * a.kper, c1 = min(nsteps, c0 + a.kper), per = (c1 - c0 + NW - 1) / NW;
        kb = SHARED ? c0 : min(c1, c0 + wave * per); ke = SHARED ? c1 : min(c1, kb + per);
    }

    // ---- Every lane works out one row of the tile (row lane % BM); whoever needs a row's position gets it by a lane
    // permutation.  First half: batch element and the request for the tile id.
    const int my_row = m0 + (lane & (BM - 1));
    const unsigned gm = (unsigned)min(my_row, rows - 1);
    const unsigned rb = fdiv(gm, a.d_Ma), rm = gm - __umul24(rb, (unsigned)a.Ma);
    const bool pixels = AM == A_MAP || (a.need_pix && a.tile_idx);      // rows are pixels of active tiles
    unsigned rp = 0; int rtile = 0;
    if (pixels) {
        const unsigned t = fdiv(rm, a.d_tt);
        rp = rm - __umul24(t, (unsigned)a.tt);
        rtile = ((const FISE_AS1 int*)a.tile_idx)[t];
    }

    // ---- weights: first stages.  LDS slot p of row r holds segment p ^ ((r >> 1) & 7) (conflict-free operand reads); a load
    // fills 8 rows, so between odd and even loads only bit 2 of the segment flips.
    const unsigned wrows = (unsigned)(GEGLU ? 2 * a.N : a.N);
    const int lrow = SHARED ? wave * 8 + lr : lr;       // this lane's row of a load
    const unsigned seg0 = (unsigned)(((lane & 7) ^ ((lrow >> 1) & 7)) * 16), seg1 = SHARED ? seg0 : seg0 ^ 64u;
    unsigned vb[BL], soff_b, bytes_b;
    const bf16_t* ptr_b;
    auto set_weights = [&](bool side, int kstep) {
        const unsigned pitch = (unsigned)(side ? a.K2 : a.K) * 2u;
        ptr_b = side ? a.w2 : a.w; bytes_b = __umul24(wrows, pitch); soff_b = (unsigned)kstep * 128u;
        const unsigned row0 = __umul24((unsigned)(by * (GEGLU ? OW : BN) + lrow), pitch);
#pragma unroll
        for (int j = 0; j < BL; ++j) {                  // GEGLU: value rows, then the gate rows N further down
            unsigned jr = (unsigned)(j * RB);
            if (GEGLU && j >= BL / 2) jr += (unsigned)(a.N - OW);
            vb[j] = row0 + (j & 1 ? seg1 : seg0) + jr * pitch;      // rows past the matrix lie past the descriptor
        }
    };
    unsigned char* const my_ring = ring + wave * (SHARED ? 1024 : NST * STAGE);      // where this wave's loads go
    int kw = kb;                                        // weight cursor
    set_weights(kb >= nsteps1, kb >= nsteps1 ? kb - nsteps1 : kb);
    auto issue_b = [&](int st) {                        // steps past the range: a descriptor of size zero, no traffic
        const __amdgpu_buffer_rsrc_t rs = buf(ptr_b, kw < ke ? bytes_b : 0u);
        unsigned char* base = my_ring + st * STAGE + BM * 128;
#pragma unroll
        for (int j = 0; j < BL; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + j * (RB * 128)), 16, vb[j], soff_b, 0, 0);
        ++kw; soff_b += 128u;
        if (AM == A_MAP && kw == nsteps1 && kw < ke) set_weights(true, 0);
    };
    // Where many row tiles share a slice of the weights they walk it in step, and each of its lines is cold for all of them at
    // once: their loads then wait for memory instead of L2.  So the row tiles first touch the slice, each a share of its lines
    // (one dword per line, into a stage that is filled later).  1536 x 320 x 2880 in 240 tiles: K loop 6.4 -> 5.0 us (85 -> 110
    // GB/s per CU); short K ranges do not earn it back.
    if (a.gx >= 12 && a.kper >= 32) {
        const int c0 = bz * a.kper, c1 = min(nsteps1, c0 + a.kper);
        const __amdgpu_buffer_rsrc_t rs = buf(a.w, bytes_b);
        if constexpr (SHARED) {
            for (int q = c0 + bx * NW + wave; q < c1; q += a.gx * NW)
#pragma unroll
                for (int r = 0; r < BN; r += 64)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)my_ring, 4,
                                                             r + lane < BN ? __umul24((unsigned)(by * BN + r + lane), (unsigned)a.K * 2u) + q * 128 : OOB, 0, 0, 0);
        } else {
        const int half = BN == 32 ? lane >> 5 : 0;
        const unsigned off = __umul24((unsigned)(by * (GEGLU ? OW : BN) + (lane & (BN - 1)) + (GEGLU && lane >= OW ? a.N - OW : 0)), (unsigned)a.K * 2u);
        constexpr int PER = BN == 32 ? 2 : 1;
        for (int q = c0 + (bx * NW + wave) * PER; q < c1; q += a.gx * NW * PER)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)my_ring, 4, off + (q + half) * 128, 0, 0, 0);
        }
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) issue_b(s);

    // ---- second half of the row: position on the output map
    unsigned ryx = rm, rpix = 0; int ry = 0, rx = 0;
    if (pixels) {
        const unsigned py = fdiv(rp, a.d_tw), ty = fdiv((unsigned)rtile, a.d_tiles_w);
        ry = (int)(__umul24(ty, (unsigned)a.tile) + py);
        rx = (int)(__umul24((unsigned)rtile - __umul24(ty, (unsigned)a.tiles_w), (unsigned)a.tile_w) + (rp - __umul24(py, (unsigned)a.tile_w)));
        ryx = __umul24((unsigned)ry, (unsigned)a.Wo) + rx;
    }
    rpix = __umul24(rb, __umul24((unsigned)a.Ho, (unsigned)a.Wo)) + ryx;

    // ---- this thread's pieces of the finished tile (four columns of a row, or four rows of a column) and their operands
    const int col0 = by * OW;
    const int sect = CONV ? 0 : (col0 >= a.sect_n) + (col0 >= 2 * a.sect_n);      // a column tile lies in one section (checked by the launcher)
    const int omode = CONV ? OUT_MAP : sect == 0 ? a.out_mode[0] : sect == 1 ? a.out_mode[1] : a.out_mode[2];
    const bool trans = !CONV && omode == OUT_TOKENS_T && a.trans4;
    int e_r[ITEMS], e_c[ITEMS], e_b[ITEMS]; unsigned e_pix[ITEMS]; bool e_ok[ITEMS];
    auto place_items = [&]() {
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int item = tid + it % IPG * NT, g0 = it / IPG * GROWS;
        e_r[it] = g0 + (trans ? (item % (GROWS / 4)) * 4 : item / CPR);
        e_c[it] = trans ? item / (GROWS / 4) : (item % CPR) * 4;
        e_ok[it] = m0 + e_r[it] < rows && col0 + e_c[it] < a.N;
        e_b[it] = __shfl((int)rb, e_r[it]);
        e_pix[it] = (unsigned)__shfl((int)rpix, e_r[it]);
    }
    };
    constexpr bool AHEAD = ITEMS <= 2;                  // more pieces per thread: placed and fetched after the K loop, all together
    u32x2_w e_bias[IPG], e_bias2[IPG], e_gate[IPG]; u32x4_w e_temb[IPG], e_res[IPG], e_ss[IPG][2][2];
    auto fetch_operands = [&](int grp) {                       // an absent operand has a descriptor of size zero: no branches, no waits
        const __amdgpu_buffer_rsrc_t s_bias = buf(a.bias, a.bias_bytes), s_bias2 = buf(a.bias2, a.bias2_bytes),
                                     s_temb = buf(a.temb, a.temb_bytes), s_res = buf(a.res, a.res_bytes);
        const int res_compact = CONV ? 0 : a.res_compact, res_shift = res_compact == 2 ? 2 : 1;       // float rows / bf16 (16 bytes are fetched either way, 8 of them used)
#pragma unroll
        for (int it = 0; it < IPG; ++it) {
            const unsigned no = e_ok[grp * IPG + it] && !trans ? 0u : OOB, col = (unsigned)(col0 + e_c[grp * IPG + it]);
            e_bias[it] = __builtin_bit_cast(u32x2_w, __builtin_amdgcn_raw_buffer_load_b64(s_bias, (col * 2u) | no, 0, 0));
            if constexpr (GEGLU) {
                e_gate[it] = __builtin_bit_cast(u32x2_w, __builtin_amdgcn_raw_buffer_load_b64(s_bias, ((col + a.N) * 2u) | no, 0, 0));
            } else {
                const unsigned r = __umul24(res_compact ? (unsigned)(m0 + e_r[grp * IPG + it]) : e_pix[grp * IPG + it], (unsigned)a.N) + col;
                if constexpr (CONV) e_res[it].xy = __builtin_bit_cast(u32x2_w, __builtin_amdgcn_raw_buffer_load_b64(s_res, (r << 1) | no, 0, 0));
                else e_res[it] = __builtin_bit_cast(u32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s_res, (r << res_shift) | no, 0, 0));
                if constexpr (AM == A_MAP) {
                    e_bias2[it] = __builtin_bit_cast(u32x2_w, __builtin_amdgcn_raw_buffer_load_b64(s_bias2, (col * 2u) | no, 0, 0));
                    e_temb[it] = __builtin_bit_cast(u32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s_temb, ((__umul24((unsigned)e_b[grp * IPG + it], (unsigned)a.temb_stride) + col) * 4u) | no, 0, 0));
                }
            }
        }
        if constexpr (!GEGLU)
#pragma unroll
            for (int v = 0; v < 2; ++v)
                if (v < a.nview) {
                    const __amdgpu_buffer_rsrc_t s = buf(a.view[v].ss, (unsigned)a.B * a.view[v].dstC * 8u);
#pragma unroll
                    for (int it = 0; it < IPG; ++it) {
                        const unsigned no = e_ok[grp * IPG + it] && !trans ? 0u : OOB;
                        const unsigned off = ((__umul24((unsigned)e_b[grp * IPG + it], (unsigned)a.view[v].dstC) + a.view[v].c_off + col0 + e_c[grp * IPG + it]) * 8u) | no;
                        e_ss[it][v][0] = __builtin_bit_cast(u32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s, off, 0, 0));
                        e_ss[it][v][1] = __builtin_bit_cast(u32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s, off, 16, 0));
                    }
                }
    };
    if constexpr (AHEAD) { place_items(); fetch_operands(0); }

    // ---- A operand
    unsigned va[AL], soff_a, bytes_a = a.src[0].bytes;
    const bf16_t* ptr_a = a.src[0].p;
    int ka = kb;                                        // cursor: K step, source, tap, channel within the source, channels of the source
    int si = 0, tap = 0, cc = 0, cn = a.C0;
    unsigned in0[AL], valid[AL], out0[AL];              // pixel under tap (0, 0) (wraps at the border), taps inside the image | parities << 16; output pixel
    if constexpr (AM == A_ROWS) {
        soff_a = (unsigned)kb * 128u;
        const unsigned row0 = (unsigned)(m0 + lrow) * a.src[0].pitch;
#pragma unroll
        for (int j = 0; j < AL; ++j) va[j] = row0 + (j & 1 ? seg1 : seg0) + (unsigned)(j * RB) * a.src[0].pitch;     // past the last row: past the descriptor
    }
    auto set_source = [&]() {                           // base and offsets of the cursor position
        si = __builtin_amdgcn_readfirstlane(si);
        ptr_a = a.src[si].p; bytes_a = a.src[si].bytes;
        const unsigned pitch = a.src[si].pitch;
        soff_a = (unsigned)cc * 2u; cn = (int)(pitch >> 1);
        if (si >= 2) {                                  // side product: the output pixel itself
#pragma unroll
            for (int j = 0; j < AL; ++j) va[j] = (__umul24(out0[j], pitch) + (j & 1 ? seg1 : seg0)) | (out0[j] & OOB);
            return;
        }
        const int ky = a.ksize == 1 ? 0 : (tap * 11) >> 5, kx = tap - ky * a.ksize;
        unsigned px[AL];
        if (a.ups) {                                    // nearest neighbour: taps step from one input pixel to the next by parity
#pragma unroll
            for (int j = 0; j < AL; ++j) px[j] = in0[j] + __umul24((((valid[j] >> 16) & 1u) + ky) >> 1, (unsigned)a.Win) + ((((valid[j] >> 17) & 1u) + kx) >> 1);
        } else {
            const unsigned delta = (unsigned)(ky * a.Win + kx);
#pragma unroll
            for (int j = 0; j < AL; ++j) px[j] = in0[j] + delta;
        }
#pragma unroll
        for (int j = 0; j < AL; ++j) va[j] = (__umul24(px[j], pitch) + (j & 1 ? seg1 : seg0)) | ((~valid[j] >> tap) << 31);
    };
    if constexpr (AM == A_MAP) {
        // pixel under tap (0, 0) and which taps lie inside the image, worked out for this lane's row, then dealt out
        const int pad = a.ksize >> 1, iy = ry * a.stride - pad, ix = rx * a.stride - pad;
        const int hh = a.Hin << a.ups, ww = a.Win << a.ups;
        unsigned vx = 0, v = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) vx |= (k < a.ksize && (unsigned)(ix + k) < (unsigned)ww ? 1u : 0u) << k;
#pragma unroll
        for (int k = 0; k < 3; ++k) v |= (k < a.ksize && (unsigned)(iy + k) < (unsigned)hh ? vx : 0u) << (k * a.ksize);
        if (my_row >= rows) v = 0;
        v |= ((unsigned)iy & 1u) << 16 | ((unsigned)ix & 1u) << 17;
        const unsigned p0 = (unsigned)((int)rb * a.Hin + (iy >> a.ups)) * (unsigned)a.Win + (unsigned)(ix >> a.ups);
        const unsigned o0 = my_row < rows ? rpix : OOB;
#pragma unroll
        for (int j = 0; j < AL; ++j) {
            in0[j] = (unsigned)__shfl((int)p0, j * RB + lrow);
            valid[j] = (unsigned)__shfl((int)v, j * RB + lrow);
            out0[j] = (unsigned)__shfl((int)o0, j * RB + lrow);
        }
        const int Cin = a.C0 + a.C1;
        if (kb < nsteps1) {
            tap = (int)fdiv((unsigned)kb, a.d_spt); cc = kb * 64 - tap * Cin;
            if (cc >= a.C0) { si = 1; cc -= a.C0; }
        } else {
            cc = (kb - nsteps1) * 64; si = 2;
            if (cc >= a.S0) { si = 3; cc -= a.S0; }
        }
        set_source();
    }
    auto issue_a = [&](int st) {
        const __amdgpu_buffer_rsrc_t rs = buf(ptr_a, ka < ke ? bytes_a : 0u);
        unsigned char* base = my_ring + st * STAGE;
#pragma unroll
        for (int j = 0; j < AL; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + j * (RB * 128)), 16, va[j], soff_a, 0, 0);
        ++ka; soff_a += 128u;
        if constexpr (AM == A_MAP) {
            cc += 64;
            if (cc >= cn) {                             // next source (a0 -> a1 -> a0 of the next tap ... -> s0 -> s1)
                cc = 0;
                if (si == 0 && a.C1) si = 1;
                else if (si < 2) { si = ka == nsteps1 ? 2 : 0; ++tap; }
                else si = 3;
                if (ka < ke) set_source();
            }
        }
    };
#pragma unroll
    for (int s = 0; s < NST; ++s) issue_a(s);

    // ---- K loop.  The accumulators hold the transposed product (lane = row, four consecutive columns per register group).
    // One copy of the body with a rotating stage offset: the launch is short, so the code it has to fetch counts.
    unsigned rd[4];                                     // LDS offset of this lane's operand fragments within 32 rows of a stage
    const unsigned rd_own = (unsigned)((lane & 31) * 128 + (((wave * 2) ^ (lane >> 5) ^ ((lane >> 1) & 7)) * 16));     // SHARED: this wave's slice of K
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) rd[ks] = (unsigned)((lane & 31) * 128 + (((ks * 2) ^ (lane >> 5) ^ ((lane >> 1) & 7)) * 16));
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    int st = 0;
    if constexpr (SHARED) {
        // Step k: the fragments of step k + 1 are requested behind the barrier that says its stage has landed for all
        // waves, the stage of step k (in registers everywhere by then) is refilled, and the matrix pipe works on step k.
        bf16x8_t f0[TM + TN], f1[TM + TN];
        auto read = [&](bf16x8_t (&f)[TM + TN], int slot) {
            const unsigned char* p = ring + slot * STAGE + rd_own;
#pragma unroll
            for (int i = 0; i < TM; ++i) f[i] = *reinterpret_cast<const bf16x8_t*>(p + i * 4096);
#pragma unroll
            for (int j = 0; j < TN; ++j) f[TM + j] = *reinterpret_cast<const bf16x8_t*>(p + (BM + j * 32) * 128);
        };
        auto step = [&](bf16x8_t (&cur)[TM + TN], bf16x8_t (&next)[TM + TN], int k) {
            const int after = st == NST - 1 ? 0 : st + 1;
            // the first NST stages were filled weights first: behind the A loads of stage i come (NST - 1 - i) stages of A loads
            if (k == kb) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NST - 2) * AL) : "memory");
            else if (NST > 3 && k == kb + 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NST > 3 ? (NST - 3) * AL + AL + BL : 0) : "memory");
            else if (NST > 4 && k == kb + 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NST > 4 ? (NST - 4) * AL + 2 * (AL + BL) : 0) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NST - 2) * (AL + BL)) : "memory");
            read(next, after);                          // past the range: zeros (loads through a descriptor of size zero)
            issue_a(st);
            issue_b(st);
            st = after;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur[TM + j], cur[i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NST - 1) * AL) : "memory");
        read(f0, 0);
#pragma unroll 1
        for (int k = kb; k < ke; k += 2) {              // always in pairs (an exit between the two costs copies of all
            step(f0, f1, k);                            // accumulators): a stage past the range holds zeros
            step(f1, f0, k + 1);
        }
    } else
#pragma unroll 1
    for (int k = kb; k < ke; ++k) {
        // The stage's loads have landed when at most the younger ones are in flight.  The first stages were filled weights
        // first, so behind the A loads of stage i come (NST - 1 - i) stages of A loads and i whole stages.
        if (k == kb) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * AL) : "memory");
        else if (NST > 2 && k == kb + 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * AL + AL + BL) : "memory");
        else if (NST > 3 && k == kb + 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NST > 3 ? (NST - 3) * AL + 2 * (AL + BL) : 0) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * (AL + BL)) : "memory");
        const unsigned char* stage = my_ring + st * STAGE;
        bf16x8_t fa[4][TM], fb[4][TN];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const unsigned char* p = stage + rd[ks];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[ks][i] = *reinterpret_cast<const bf16x8_t*>(p + i * 4096);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[ks][j] = *reinterpret_cast<const bf16x8_t*>(p + (BM + j * 32) * 128);
        }
        // The stage is refilled as soon as its fragments are in registers: NST stages stay in flight while the matrix
        // pipe works (refilled one step later, a two-stage ring leaves the memory idle while a stage is read).
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue_a(st);
        issue_b(st);
        st = st == NST - 1 ? 0 : st + 1;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // the loads past the end of the range still target the ring
    __syncthreads();
    if constexpr (!AHEAD) { place_items(); fetch_operands(0); }
    float* const part = reinterpret_cast<float*>(ring);
    f32x4_w v[ITEMS], g[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) v[it] = g[it] = f32x4_w{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int grp = 0; grp < GROUPS; ++grp) {
        if (grp) __syncthreads();
#pragma unroll
        for (int i = 0; i < TM / GROUPS; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x16_t& c = acc[grp * (TM / GROUPS) + i][j];
                    *reinterpret_cast<f32x4_w*>(&part[(wave * GROWS + i * 32 + (lane & 31)) * PITCH + j * 32 + q * 8 + (lane >> 5) * 4]) =
                        f32x4_w{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                }
        __syncthreads();
        if (trans) {
#pragma unroll
            for (int it = grp * IPG; it < (grp + 1) * IPG; ++it)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float* p = &part[(w * GROWS + e_r[it] - grp * GROWS) * PITCH + e_c[it]];
                    v[it] += f32x4_w{p[0], p[PITCH], p[2 * PITCH], p[3 * PITCH]};
                }
        } else {
#pragma unroll
            for (int it = grp * IPG; it < (grp + 1) * IPG; ++it)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float* p = &part[(w * GROWS + e_r[it] - grp * GROWS) * PITCH + e_c[it]];
                    v[it] += *reinterpret_cast<const f32x4_w*>(p);
                    if (GEGLU) g[it] += *reinterpret_cast<const f32x4_w*>(p + OW);
                }
        }
    }
    if (a.splits > 1) {
        // park the tile (16 bytes per lane, written through to memory), count this workgroup; the last one goes on
        constexpr int SLOT = (GEGLU ? 2 : 1) * BM * OW * 4;
        const unsigned tile = (unsigned)(by * a.gx + bx), base = tile * a.splits;
        const __amdgpu_buffer_rsrc_t s_part = buf(a.partial, (unsigned)IGEMM_PARTIAL_BYTES);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const unsigned off = (base + bz) * SLOT + (unsigned)(it * NT + tid) * 16u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_w, v[it]), s_part, off, 0, 17);
            if (GEGLU) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_w, g[it]), s_part, off + BM * OW * 4, 0, 17);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int* const flag = reinterpret_cast<int*>(ring + NW * GROWS * PITCH * 4 - 4);      // the last pad word of the partial tiles
        if (tid == 0) {
            const int old = __hip_atomic_fetch_add(a.counters + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (old == a.splits - 1) __hip_atomic_store(a.counters + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *flag = old;
        }
        __syncthreads();
        if (*flag != a.splits - 1) return;
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) v[it] = g[it] = f32x4_w{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int z = 0; z < a.splits; ++z) {            // split order, whoever is last
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const unsigned off = (base + z) * SLOT + (unsigned)(it * NT + tid) * 16u;
                v[it] += __builtin_bit_cast(f32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s_part, off, 0, 17));
                if (GEGLU) g[it] += __builtin_bit_cast(f32x4_w, __builtin_amdgcn_raw_buffer_load_b128(s_part, off + BM * OW * 4, 0, 17));
            }
        }
    }

    // ---- epilogue: sum, biases, gate, then time projection + residual as one term; stores
    bf16_t* const outp = sect == 0 ? a.out[0] : sect == 1 ? a.out[1] : a.out[2];
    const int scol0 = col0 - sect * a.sect_n;
    if constexpr (CONV) {
        // A group's results are packed in registers, the next group's operands requested, and only then stored: behind the
        // stores the loads would wait for them.
#pragma unroll
        for (int grp = 0; grp < GROUPS; ++grp) {
            u32x2_w y[IPG], yv[IPG][2];
#pragma unroll
            for (int it = 0; it < IPG; ++it) {
                const f32x4_w sum = v[grp * IPG + it];
                float x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    auto part = [q](const u32x2_w& w) { return q & 1 ? hi16(w[q >> 1]) : lo16(w[q >> 1]); };
                    const float res = part(u32x2_w{e_res[it][0], e_res[it][1]});
                    x[q] = sum[q] + part(e_bias[it]);
                    x[q] += part(e_bias2[it]);
                    x[q] += res + __uint_as_float(e_temb[it][q]);
                }
                y[it] = u32x2_w{f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (i < a.nview) {                  // as put_views4
                        float u[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const u32x4_w& ss = e_ss[it][i][q >> 1];
                            u[q] = fmaf(q & 1 ? hi16(y[it][q >> 1]) : lo16(y[it][q >> 1]), __uint_as_float(ss[(q & 1) * 2]), __uint_as_float(ss[(q & 1) * 2 + 1]));
                        }
                        if (a.view[i].silu) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) u[q] = silu_f(u[q]);
                        }
                        yv[it][i] = u32x2_w{f2bf2(u[0], u[1]), f2bf2(u[2], u[3])};
                    }
            }
            if (grp + 1 < GROUPS) fetch_operands(grp + 1);
#pragma unroll
            for (int it = 0; it < IPG; ++it) {
                const int e = grp * IPG + it;
                if (!e_ok[e]) continue;
                *(FISE_AS1 u32x2_w*)(outp + (size_t)e_pix[e] * a.N + col0 + e_c[e]) = y[it];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (i < a.nview) *(FISE_AS1 u32x2_w*)(a.view[i].dst + (size_t)e_pix[e] * a.view[i].dstC + a.view[i].c_off + col0 + e_c[e]) = yv[it][i];
            }
        }
        return;
    }
    if (trans) {
        const unsigned HW = (unsigned)(a.Ho * a.Wo);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (!e_ok[it]) continue;
            FISE_AS1 bf16_t* q = (FISE_AS1 bf16_t*)(outp + ((size_t)e_b[it] * a.sect_n + scol0 + e_c[it]) * HW + (e_pix[it] - (unsigned)e_b[it] * HW));
            *(FISE_AS1 u32x2_w*)q = u32x2_w{f2bf2(v[it][0], v[it][1]), f2bf2(v[it][2], v[it][3])};
        }
        return;
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int gi = it % IPG;
        if (GROUPS > 1 && it && gi == 0) fetch_operands(it / IPG);
        float x[4] = {v[it][0] + lo16(e_bias[gi][0]), v[it][1] + hi16(e_bias[gi][0]), v[it][2] + lo16(e_bias[gi][1]), v[it][3] + hi16(e_bias[gi][1])};
        if constexpr (GEGLU) {
            x[0] *= gelu_f(g[it][0] + lo16(e_gate[gi][0])); x[1] *= gelu_f(g[it][1] + hi16(e_gate[gi][0]));
            x[2] *= gelu_f(g[it][2] + lo16(e_gate[gi][1])); x[3] *= gelu_f(g[it][3] + hi16(e_gate[gi][1]));
        } else {
            const u32x4_w w = e_res[gi];
            f32x4_w r = a.res_compact == 2 ? __builtin_bit_cast(f32x4_w, w) : f32x4_w{lo16(w[0]), hi16(w[0]), lo16(w[1]), hi16(w[1])};
            if constexpr (AM == A_MAP) {
                x[0] += lo16(e_bias2[gi][0]); x[1] += hi16(e_bias2[gi][0]); x[2] += lo16(e_bias2[gi][1]); x[3] += hi16(e_bias2[gi][1]);
                r += __builtin_bit_cast(f32x4_w, e_temb[gi]);
            }
            x[0] += r[0]; x[1] += r[1]; x[2] += r[2]; x[3] += r[3];
        }
        if (!e_ok[it]) continue;
        const int scol = scol0 + e_c[it];
        const size_t gm = (size_t)(m0 + e_r[it]);
        if (omode == OUT_TOKENS_T) {
            const size_t HW = (size_t)a.Ho * a.Wo;
            FISE_AS1 bf16_t* q = (FISE_AS1 bf16_t*)(outp + ((size_t)e_b[it] * a.sect_n + scol) * HW + (e_pix[it] - (unsigned)e_b[it] * (unsigned)HW));
#pragma unroll
            for (int t = 0; t < 4; ++t) q[t * HW] = f2bf(x[t]);
            continue;
        }
        const u32x2_w packed = {f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
        if (omode == OUT_COMPACT_F32) {
            if (outp) *(FISE_AS1 f32x4_w*)(reinterpret_cast<float*>(outp) + gm * a.sect_n + scol) = f32x4_w{x[0], x[1], x[2], x[3]};
            if (a.mirror) *(FISE_AS1 u32x2_w*)(a.mirror + gm * a.sect_n + scol) = packed;
        } else if (omode == OUT_COMPACT) {
            *(FISE_AS1 u32x2_w*)(outp + gm * a.sect_n + scol) = packed;
        } else {
            *(FISE_AS1 u32x2_w*)(outp + (size_t)e_pix[it] * a.sect_n + scol) = packed;
            if (!GEGLU && a.nview) {
                ViewSS ss;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) { ss.s[i][q] = __uint_as_float(e_ss[gi][i][0][q]); ss.s[i][4 + q] = __uint_as_float(e_ss[gi][i][1][q]); }
                put_views4(a.view, a.nview, e_pix[it], scol, x, ss);
            }
        }
    }
#endif
}

__global__ void zero_ints_kernel(int* p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Derived fields of the argument block: divisors, operand sizes, what the epilogue addresses.
static void prepare(IgemmArgs& a, int ncols) {
    const int rows = a.B * a.Ma;
    if (a.tile_w <= 0) a.tile_w = a.tile;
    a.need_pix = a.res && a.res_compact == 0;
    bool tokens_t = false;
    for (int s = 0; s < a.nsect; ++s) { a.need_pix |= a.out_mode[s] == OUT_MAP || a.out_mode[s] == OUT_TOKENS_T; tokens_t |= a.out_mode[s] == OUT_TOKENS_T; }
    // four consecutive rows are four consecutive pixels of a map row (or tokens) at an offset that is a multiple of 4
    const bool runs = a.tile_idx ? a.tile_w % 4 == 0 && a.Wo % 4 == 0 : a.Ma % 4 == 0 && (a.Ho * a.Wo) % 4 == 0;
    a.trans4 = tokens_t && runs && a.Ma % 4 == 0 && !a.bias && !a.bias2 && !a.temb && !a.res && !a.geglu;
    a.tt = a.tile * a.tile_w;
    a.d_gx = fast_div(a.gx); a.d_gy = fast_div(a.gy); a.d_Ma = fast_div(a.Ma); a.d_tt = fast_div(a.tt); a.d_tw = fast_div(a.tile_w);
    a.d_tiles_w = fast_div(a.tiles_w); a.d_spt = fast_div((a.C0 + a.C1) / 64);
    const unsigned n_in = a.a_compact ? (unsigned)rows : (unsigned)(a.B * a.Hin * a.Win), n_out = (unsigned)(a.B * a.Ho * a.Wo);
    a.src[0].p = a.a0; a.src[0].pitch = 2u * a.C0; a.src[1].p = a.a1; a.src[1].pitch = 2u * a.C1;
    a.src[2].p = a.s0; a.src[2].pitch = 2u * a.S0; a.src[3].p = a.s1; a.src[3].pitch = 2u * a.S1;
    a.bias_bytes = a.bias ? 2u * ncols : 0u; a.bias2_bytes = a.bias2 ? 2u * a.N : 0u;
    a.temb_bytes = a.temb ? 4u * ((a.B - 1) * a.temb_stride + a.N) : 0u;
    a.res_bytes = !a.res ? 0u : (a.res_compact == 0 ? n_out : (unsigned)rows) * (unsigned)a.N * (a.res_compact == 2 ? 4u : 2u);
    for (int i = 0; i < 4; ++i) a.src[i].bytes = (i < 2 ? n_in : n_out) * a.src[i].pitch;
}

template <int TM, int TN, int NST, int AM, bool GEGLU, bool SHARED = false>
static int launch_tile(const IgemmArgs& a, hipStream_t st) {
    constexpr int NW = 4, lds = (SHARED ? 1 : NW) * NST * (32 * TM + 32 * TN) * 128;
    // raised once per instantiation (initialisation of a function-local static is thread safe)
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wave_gemm_kernel<TM, TN, NW, NST, AM, GEGLU, SHARED>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "wave gemm: cannot raise the dynamic LDS limit");
    const double rows = (double)a.B * a.Ma, ncols = a.geglu ? 2.0 * a.N : a.N, K = (double)a.K + a.K2;
    {
        ProfileScope prof(GEGLU ? PROF_IGEMM_GEGLU : AM == A_MAP ? PROF_IGEMM : PROF_ROWS_GEMM, 2.0 * rows * ncols * K, 2.0 * (ncols * K + rows * (a.C0 + a.C1 + a.S0 + a.S1) + rows * a.N), st);
        hipLaunchKernelGGL((wave_gemm_kernel<TM, TN, NW, NST, AM, GEGLU, SHARED>), dim3((unsigned)(a.gx * a.gy * a.splits)), dim3(64 * NW), lds, st, a);
    }
    FISE_CHECK_LAUNCH("wave gemm");
    return FISE_OK;
}

static bool wave_gemm_fits(const IgemmArgs& a) {
    const int rows = a.B * a.Ma;
    constexpr size_t kLim = (size_t)1 << 31;            // 32-bit buffer offsets, top bit reserved for "no such row"
    if (a.pro != PRO_NONE || a.C0 % 64 || a.C1 % 64 || a.S0 % 64 || a.S1 % 64 || a.N % 4) return false;
    if (a.nsect > 1 && a.sect_n % 64) return false;     // a column tile has one destination
    if (a.geglu && (!a.a_compact || a.nsect != 1 || a.temb || a.res || a.nview || a.bias2)) return false;
    if (!a.a_compact && !a.tile_idx) return false;
    const size_t npix_in = a.a_compact ? (size_t)rows : (size_t)a.B * a.Hin * a.Win, npix_out = (size_t)a.B * a.Ho * a.Wo;
    const size_t ncols = a.geglu ? 2 * (size_t)a.N : (size_t)a.N;
    if (npix_in >= 1u << 24 || npix_out >= 1u << 24 || rows >= 1 << 24) return false;   // 24-bit multiplies
    if (a.a_compact && (a.temb || a.bias2)) return false;      // epilogue terms of the convolutions only
    return npix_in * std::max(a.C0, a.C1) * 2 < kLim && npix_out * std::max({a.S0, a.S1, a.N}) * 2 < kLim &&
           ncols * std::max(a.K, a.K2) * 2 < kLim && (size_t)rows * a.N * 4 < kLim;
}

// Compact rows of one section from here on: igemm.hip's 64 x 128 and 64 x 64 tiles (8192 x 320 x 320 12.8 against 14.3 us,
// 2048 x 640 x 640 12.7 against 13.3 us on shared tiles).
constexpr int BLOCK_ROWS = 2048;
bool wave_gemm_takes(const IgemmArgs& a) {
    return wave_gemm_fits(a) && (a.B * a.Ma < BLOCK_ROWS || !a.a_compact || a.geglu || a.nsect > 1);
}

// Tile and K split of a launch: the cheapest of the combinations under times measured per part of a launch (us, from time
// stamps inside the kernel and kernel traces over the shapes of steps and dense builds).
//  - PRIVATE, a ring per wave, 256 workgroups at once.  `fixed`: start, row positions, first loads, sum over the waves,
//    epilogue, and the gap to the launch before.  `iter`: four K steps, one per wave (operands at the 71 - 88 GB/s a CU gets with all busy).
//  - SHARED, 64 x 64 on one ring of 48 KB: every wave multiplies a 16-deep slice of each K step over the whole tile, so a
//    staged byte is read once, and three workgroups per CU hide each other's start and epilogue, which many tiles of
//    a short K consist of: `tile` + `iter` per K step of a tile and CU.  5504 x 320 x 2880 36 -> 24 us (64 x 128 tiles of
//    eight waves that read a staged byte 2.7 times), 1376 x 1920 x 640 23 -> 15, with GEGLU 1376 x 5120 x 640 39 -> 26 us.
//    Beyond ~96 K steps (`iter_long`) the workgroups of an XCD drift apart and fall out of its L2.
//  - BLOCK, 64 x 160 on one ring of 112 KB: 1/46 of an operand row per product instead of 1/32, one workgroup per CU and a
//    long epilogue (ten pieces per thread): 8192 x 320 x 9600 105 (SHARED) -> 64 us, 2048 x 640 x 11520 with 1x1 side product 76
//    -> 54 us.  Widths of a 320-channel UNet are multiples of 160: no columns to spare.
// A K split over workgroups adds parking, counting and re-reading the tiles (`park`, `park_s` per split).
// Held against every tile and split on the 164 ResNet convolutions of a 64 x 64 x 320 / 32 x 32 x 640 / 16 x 16 x 1280 UNet with
// 32 to 8192 rows and cold weights, the choice is 4 % from the best on average.  It is furthest off at 90 - 180 K steps and ~160 tiles
// of 64 x 64, where it takes BLOCK in four splits or SHARED in two (2048 x 320 x 8640: 39 us, PRIVATE unsplit 29; 512 x 1280 x 5760:
// 34 and 27): fewer than 256 workgroups get more per CU than `iter` says, and four parked BLOCK tiles cost more than `park`.
enum { PRIVATE = 0, SHARED_RING = 1, BLOCK = 2 };
struct TileShape { int kind, tm, tn; double fixed, tile, iter, iter_long, park, park_s; };
static const TileShape kShapes[] = {
    {PRIVATE, 1, 1, 4.3, 0.0, 0.39, 0.39, 2.0, 0.15}, {PRIVATE, 1, 2, 4.8, 0.0, 0.56, 0.56, 2.3, 0.3}, {PRIVATE, 2, 2, 5.8, 0.0, 0.92, 0.92, 3.2, 0.6},
    {SHARED_RING, 2, 2, 5.2, 1.2, 0.235, 0.32, 3.2, 0.6}, {BLOCK, 2, 5, 13.0, 0.0, 0.4, 0.4, 4.0, 1.5}};

int launch_wave_gemm(IgemmArgs a, const IgemmWorkspace* ws, hipStream_t st) {
    const int rows = a.B * a.Ma, ncols = a.geglu ? 2 * a.N : a.N, nsteps = (a.K + a.K2) / 64;
    int kind = PRIVATE, best_tm = 1, best_tn = 1, best_s = 1; double best = 1e30;
    const int max_s = ws && ws->counters && ws->partial ? 8 : 1;
    for (const TileShape& sh : kShapes) {
        if (a.geglu && sh.tn == 1) continue;
        if (sh.kind == BLOCK && (a.a_compact || a.N % 160 || a.nsect > 1 || a.out_mode[0] != OUT_MAP || (a.res && a.res_compact))) continue;
        const int gx = ceil_div(rows, 32 * sh.tm), gy = ceil_div(ncols, 32 * sh.tn);
        for (int s = 1; s <= max_s; ++s) {
            const int per = ceil_div(nsteps, s);
            if (s > 1 && (per < 4 || ceil_div(nsteps, per) != s)) continue;
            if (s > 1 && ((long long)gx * gy > IGEMM_COUNTERS || (size_t)gx * gy * s * 32 * sh.tm * 32 * sh.tn * 4 > ws->partial_bytes)) break;
            const long long n = (long long)gx * gy * s;
            const double iter = nsteps > 96 ? sh.iter_long : sh.iter;
            double t = s > 1 ? sh.park + sh.park_s * s : 0.0;
            if (sh.kind == SHARED_RING) t += sh.fixed + std::max(1.0, n / 256.0) * (sh.tile + per * iter);
            else t += (double)((n + 255) / 256) * (sh.fixed + (sh.kind == PRIVATE ? ceil_div(per, 4) : per) * iter);
            if (t < best) { best = t; kind = sh.kind; best_tm = sh.tm; best_tn = sh.tn; best_s = s; }
        }
    }
    a.splits = best_s; a.kper = ceil_div(nsteps, best_s);
    a.gx = ceil_div(rows, 32 * best_tm); a.gy = ceil_div(ncols, 32 * best_tn);
    prepare(a, ncols);
    if (a.splits > 1) {
        a.partial = ws->partial; a.counters = ws->counters;
        if (!ws->counters_zeroed) {                     // once per call: every launch leaves its counters at zero
            hipLaunchKernelGGL(zero_ints_kernel, dim3(ceil_div(IGEMM_COUNTERS, 256)), dim3(256), 0, st, ws->counters, IGEMM_COUNTERS);
            FISE_CHECK_LAUNCH("zero counters");
            ws->counters_zeroed = true;
        }
    }
    int e;
    if (kind == BLOCK) e = launch_tile<2, 5, 4, A_MAP, false, true>(a, st);
    else if (kind == SHARED_RING)
        e = a.geglu ? launch_tile<2, 2, 3, A_ROWS, true, true>(a, st) : a.a_compact ? launch_tile<2, 2, 3, A_ROWS, false, true>(a, st) : launch_tile<2, 2, 3, A_MAP, false, true>(a, st);
    else if (a.geglu) e = best_tm == 1 ? launch_tile<1, 2, 2, A_ROWS, true>(a, st) : launch_tile<2, 2, 2, A_ROWS, true>(a, st);
    else if (a.a_compact)
        e = best_tm == 2 ? launch_tile<2, 2, 2, A_ROWS, false>(a, st) : best_tn == 2 ? launch_tile<1, 2, 2, A_ROWS, false>(a, st) : launch_tile<1, 1, 2, A_ROWS, false>(a, st);
    else
        e = best_tm == 2 ? launch_tile<2, 2, 2, A_MAP, false>(a, st) : best_tn == 2 ? launch_tile<1, 2, 2, A_MAP, false>(a, st) : launch_tile<1, 1, 2, A_MAP, false>(a, st);
    if (e) return e;
    if (a.ln_out) {
        if (a.nsect != 1 || a.out_mode[0] != OUT_COMPACT_F32 || a.geglu || !a.ln_gamma || !a.ln_beta)
            return fail(FISE_ERR_SHAPE, "igemm: LayerNorm output needs one float compact section");
        return launch_ln_rows(a.out[0], 1, rows, a.N, a.ln_gamma, a.ln_beta, a.ln_eps, a.ln_out, nullptr, 1, 1, 1, 1, 1, st);
    }
    return FISE_OK;
}

}  // namespace fise
