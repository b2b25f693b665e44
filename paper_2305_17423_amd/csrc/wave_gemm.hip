// Gathered GEMM for tiles of 32 or 64 rows whose K loop is split over the waves of ONE workgroup.
//
//   out[row, n] = epilogue( sum_k A[row, k] * W[n, k]  (+ sum_k A2[row, k] * W2[n, k]) )      (see igemm.h)
//
// What bounds the masked step is not bandwidth or MFMA rate but the fixed cost of some 200 dependent launches (half of them this
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
#include <type_traits>
#include "igemm.h"
#include "patch.h"
#include "profile.h"

namespace fise {

enum { A_ROWS = 0, A_MAP = 1 };         // compact rows / pixels of maps (taps, two sources, side product)

// ---- PATCH form (3x3, stride 1, square tiles of edge 2, 4 or 8): the pixels of a tile and their ring are brought into LDS once for 64
// channels and read under all nine taps; the weights run through a ring of their own, a kernel row at a time.  Bound by the LDS-direct
// loads (36 KB of weights and 8 - 32 KB of patches per chunk and column tile of 32; 0.42 us at the 125 GB/s of a CU, 0.6 - 0.7 measured)
// and, from 20 chunks of 1280 wide layers on, by their cold weights.
// Loads a lane issues in the steps u0 <= u < u1 (three per chunk): every step LB weight loads, the first one before them SLOTS patch loads.
constexpr int patch_loads(int u0, int u1, int LB, int SLOTS) {
    int n = 0;
    for (int u = u0; u < u1; ++u) n += LB + ((u + 3000) % 3 == 0 ? SLOTS : 0);
    return n;
}
constexpr int patch_min(int a, int b) { return a < b ? a : b; }
// Loads that may be in flight when the operands of step s + 1 have to be there (s = ky of any chunk): the weights of step t went
// out in step t - AHEAD, the patch of chunk c in step 3 (c - NPB + 1) in front of that step's weights.
constexpr int patch_flight(int s, int AHEAD, int NPB, int LB, int SLOTS) {
    const int w = patch_loads(s + 2 - AHEAD, s, LB, SLOTS);
    return (s + 1) % 3 ? w : patch_min(w, LB + patch_loads(s + 5 - 3 * NPB, s, LB, SLOTS));
}
// The same in front of step 0, when the steps below 0 have gone out (those below -AHEAD without weights).
constexpr int patch_flight0(int AHEAD, int NPB, int LB, int SLOTS) {
    const int a0 = 3 - 3 * NPB, a = a0 >= -AHEAD ? LB + patch_loads(a0 + 1, 0, LB, SLOTS) : patch_loads(-AHEAD, 0, LB, SLOTS);
    return patch_min(patch_loads(1 - AHEAD, 0, LB, SLOTS), a);
}

// What the products of a group differ in.
struct Product { const bf16_t* w; int N, sect_n; bf16_t* out0; int mode0; };

// SHARED: one ring for the workgroup instead of one per wave; which form a launch takes is gemm_choice.h's rule.

template <int TM, int TN, int NW, int NST, int AM, bool GEGLU, bool SHARED, int PATCH = 0, int NPB = 0>
__device__ __forceinline__ void wave_gemm_tile(const IgemmArgs& a, const Product& pr, const int bx, const int by, const int bz) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 32 * TM, BN = 32 * TN, NT = 64 * NW;
    constexpr int RB = SHARED ? 8 * NW : 8;             // rows between two loads of a lane (one load of a wave fills 8 rows of 128 bytes)
    constexpr int AL = BM / RB, BL = BN / RB;           // 16-byte loads per lane and K step
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int PITCH = BN + 4;                       // floats per row of a partial tile in LDS
    constexpr int OW = GEGLU ? BN / 2 : BN;             // output columns of the tile
    constexpr int GROUPS = SHARED && !PATCH ? TM : 1, GROWS = BM / GROUPS;       // the waves' sums are finished in groups of rows: what fits in the ring
    constexpr int CPR = OW / 4, IPG = GROWS * CPR / NT, ITEMS = GROUPS * IPG;      // four-column pieces per row, per thread and group, per thread
    constexpr unsigned OOB = 0x80000000u;               // beyond every descriptor: the load returns zeros
    using PG = Patch<BM, PATCH ? PATCH : 8>;
    constexpr int LB = 3 * BL, WSTAGE = 3 * BN * 128, NB = NST;       // PATCH: weight loads per lane and step, bytes of a step's weights, steps in LDS
    static_assert(GROWS * CPR % NT == 0 && (PATCH ? NPB * PG::BYTES + NB * WSTAGE : (SHARED ? 1 : NW) * NST * STAGE) >= NW * GROWS * PITCH * 4, "tile");
    static_assert(!PATCH || (SHARED && AM == A_MAP && BM <= 64 && TM + BL <= LB && NB >= 4 && NPB >= 2 && NPB <= 3), "patch form");
    constexpr bool CONV = TN == 5 || PATCH;             // one map out, bf16 map as residual
    static_assert(!SHARED || (NW == 4 && NST >= 3), "a shared stage has one 16-deep slice of K per wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];      // [NW or 1][NST][STAGE], later [NW][GROWS][PITCH] floats

    // Kernel arguments arrive through scalar loads placed where a field is first used; named here they come as one batch.
    asm volatile("" ::"s"(a.kper), "s"(a.d_Ma.mul), "s"(a.d_tt.mul),
                 "s"(a.d_tw.mul), "s"(a.d_tiles_w.mul), "s"(a.B), "s"(a.Ma), "s"(a.K), "s"(a.K2), "s"(pr.N), "s"(pr.w), "s"(a.tile_idx), "s"(a.need_pix));
    asm volatile("" ::"s"(a.Ho), "s"(a.Wo), "s"(a.tile), "s"(pr.sect_n), "s"(pr.mode0), "s"(a.bias), "s"(a.bias_bytes), "s"(a.temb), "s"(a.temb_bytes),
                 "s"(a.res), "s"(a.res_bytes), "s"(a.res_compact), "s"(a.nview), "s"(a.src[0].p), "s"(a.src[0].bytes));
    if constexpr (AM == A_MAP) asm volatile("" ::"s"(a.Hin), "s"(a.Win), "s"(a.ksize), "s"(a.stride), "s"(a.ups), "s"(a.C0), "s"(a.d_spt.mul), "s"(a.bias2), "s"(a.bias2_bytes));
    const int tid = threadIdx.x, lane = tid & 63, lr = lane >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
    const unsigned wrows = (unsigned)(GEGLU ? 2 * pr.N : pr.N);
    const int lrow = SHARED ? wave * 8 + lr : lr;       // this lane's row of a load
    const unsigned seg0 = (unsigned)(((lane & 7) ^ ((lrow >> 1) & 7)) * 16), seg1 = SHARED ? seg0 : seg0 ^ 64u;
    unsigned vb[BL], soff_b, bytes_b;
    const bf16_t* ptr_b;
    auto set_weights = [&](bool side, int kstep) {
        const unsigned pitch = (unsigned)(side ? a.K2 : a.K) * 2u;
        ptr_b = side ? a.w2 : pr.w; bytes_b = __umul24(wrows, pitch); soff_b = (unsigned)kstep * 128u;
        const unsigned row0 = __umul24((unsigned)(by * (GEGLU ? OW : BN) + lrow), pitch);
#pragma unroll
        for (int j = 0; j < BL; ++j) {                  // GEGLU: value rows, then the gate rows N further down
            unsigned jr = (unsigned)(j * RB);
            if (GEGLU && j >= BL / 2) jr += (unsigned)(pr.N - OW);
            vb[j] = row0 + (j & 1 ? seg1 : seg0) + jr * pitch;      // rows past the matrix lie past the descriptor
        }
    };
    unsigned char* const my_ring = ring + wave * (SHARED ? 1024 : NST * STAGE);      // where this wave's loads go
    int kw = kb;                                        // weight cursor
    if constexpr (PATCH) set_weights(false, 0); else set_weights(kb >= nsteps1, kb >= nsteps1 ? kb - nsteps1 : kb);
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
    if (!PATCH && a.gx >= 12 && a.kper >= 32) {
        const int c0 = bz * a.kper, c1 = min(nsteps1, c0 + a.kper);
        const __amdgpu_buffer_rsrc_t rs = buf(pr.w, bytes_b);
        if constexpr (SHARED) {
            for (int q = c0 + bx * NW + wave; q < c1; q += a.gx * NW)
#pragma unroll
                for (int r = 0; r < BN; r += 64)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)my_ring, 4,
                                                             r + lane < BN ? __umul24((unsigned)(by * BN + r + lane), (unsigned)a.K * 2u) + q * 128 : OOB, 0, 0, 0);
        } else {
        const int half = BN == 32 ? lane >> 5 : 0;
        const unsigned off = __umul24((unsigned)(by * (GEGLU ? OW : BN) + (lane & (BN - 1)) + (GEGLU && lane >= OW ? pr.N - OW : 0)), (unsigned)a.K * 2u);
        constexpr int PER = BN == 32 ? 2 : 1;
        for (int q = c0 + (bx * NW + wave) * PER; q < c1; q += a.gx * NW * PER)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)my_ring, 4, off + (q + half) * 128, 0, 0, 0);
        }
    }
    // PATCH: chunks of 64 channels [ch0, ch1) of the main product, K steps [sd0, sd1) of the side product; a step is the three
    // taps of a kernel row or one K step of the side product.
    const int nchunk = nsteps1 / 9;
    const int ch0 = min(nchunk, bz * a.kper), ch1 = min(nchunk, ch0 + a.kper), nmain = 3 * (ch1 - ch0);
    const int sd0 = min(nsteps - nsteps1, bz * a.kper2), nside = min(nsteps - nsteps1, sd0 + a.kper2) - sd0;
    unsigned char* const wring = ring + NPB * PG::BYTES;       // [NB][WSTAGE] behind the patches [NPB][PG::BYTES]
    unsigned va_s[TM], vb_s[BL], out_s[TM]; const bf16_t* ptr_s = nullptr; unsigned bytes_s = 0, soff_s = 0, end_s = 0, soff_w2 = 0;    // side product: rows, weights, cursor
    int vstep = 0, vky = 0; unsigned wslot = 0;                // next step to request, its kernel row, its place in the ring
    const unsigned tap_bytes = (unsigned)(a.C0 + a.C1) * 2u;
    if constexpr (PATCH) {
        soff_b = (unsigned)ch0 * 128u;
        // The same first touch as above: line q of a row of W is tap q / chunks, chunk q % chunks of this range.
        if (a.touch) {
            const __amdgpu_buffer_rsrc_t rs = buf(pr.w, bytes_b);
            const int nch = ch1 - ch0, lines = 9 * nch;
            const unsigned off = __umul24((unsigned)(by * BN + (lane & (BN - 1))), (unsigned)a.K * 2u) + soff_b;
            constexpr int PER = 64 / BN;
            for (int q = (bx * NW + wave) * PER; q < lines; q += a.gx * NW * PER) {
                const int l = q + (PER == 2 ? lane >> 5 : 0), t = l / nch;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(wring + wave * 1024), 4, l < lines ? off + t * tap_bytes + (l - t * nch) * 128 : OOB, 0, 0, 0);
            }
        }
    }
    auto set_side = [&](int cc2) {                             // source of the side product that holds channel cc2
        const int i = cc2 >= a.S0 ? 3 : 2;
        ptr_s = a.src[i].p; bytes_s = a.src[i].bytes; end_s = a.src[i].pitch; soff_s = (unsigned)(cc2 - (i == 3 ? a.S0 : 0)) * 2u;
#pragma unroll
        for (int l = 0; l < TM; ++l) va_s[l] = (__umul24(out_s[l], end_s) + seg0) | (out_s[l] & OOB);
    };
    // weights of the next step into its ring slot; behind the main product the rows of A and W of a side step.  LB loads always.
    auto issue_step = [&]() {
        unsigned char* base = wring + wslot + wave * 1024;
        if (vstep < nmain) {
            const __amdgpu_buffer_rsrc_t rs = buf(pr.w, bytes_b);
#pragma unroll
            for (int l = 0; l < LB; ++l)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + l * 4096), 16, vb[l % BL], soff_b + (l / BL) * tap_bytes, 0, 0);
            soff_b += 3 * tap_bytes;
            if (++vky == 3) { vky = 0; soff_b += 128u - 9 * tap_bytes; }
        } else {
            const bool live = vstep < nmain + nside;
            const __amdgpu_buffer_rsrc_t rs = buf(ptr_s, live ? bytes_s : 0u), rw = buf(a.w2, live ? __umul24((unsigned)pr.N, (unsigned)a.K2 * 2u) : 0u);
#pragma unroll
            for (int l = 0; l < LB; ++l) {
                if (l < TM) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + l * 4096), 16, va_s[l], soff_s, 0, 0);
                else __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(base + l * 4096), 16, l < TM + BL ? vb_s[(l - TM) % BL] : OOB, soff_w2, 0, 0);
            }
            soff_s += 128u; soff_w2 += 128u;
            if (soff_s == end_s && vstep + 1 < nmain + nside) set_side(a.S0);
        }
        ++vstep;
        wslot = wslot == (NB - 1) * WSTAGE ? 0u : wslot + WSTAGE;
    };
    constexpr int FIRST_A = 3 - 3 * NPB, WAHEAD = NB - 1;      // step (before the first) in which the first patch goes out; steps the weights run ahead
    if constexpr (PATCH) {
#pragma unroll
        for (int s = -WAHEAD; s < FIRST_A; ++s) issue_step();
    } else {
#pragma unroll
        for (int s = 0; s < NST; ++s) issue_b(s);
    }

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
    const int sect = CONV ? 0 : (col0 >= pr.sect_n) + (col0 >= 2 * pr.sect_n);      // a column tile lies in one section (checked by the launcher)
    const int omode = CONV ? OUT_MAP : sect == 0 ? pr.mode0 : sect == 1 ? a.out_mode[1] : a.out_mode[2];
    const bool trans = !CONV && omode == OUT_TOKENS_T && a.trans4;
    int e_r[ITEMS], e_c[ITEMS], e_b[ITEMS]; unsigned e_pix[ITEMS]; bool e_ok[ITEMS];
    auto place_items = [&]() {
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int item = tid + it % IPG * NT, g0 = it / IPG * GROWS;
        e_r[it] = g0 + (trans ? (item % (GROWS / 4)) * 4 : item / CPR);
        e_c[it] = trans ? item / (GROWS / 4) : (item % CPR) * 4;
        e_ok[it] = m0 + e_r[it] < rows && col0 + e_c[it] < pr.N;
        e_b[it] = __shfl((int)rb, e_r[it]);
        e_pix[it] = (unsigned)__shfl((int)rpix, e_r[it]);
    }
    };
    constexpr bool AHEAD = ITEMS <= 2;                  // more pieces per thread: placed and fetched after the K loop, all together
    u32x2_t e_bias[IPG], e_bias2[IPG], e_gate[IPG]; u32x4_t e_temb[IPG], e_res[IPG], e_ss[IPG][2][2];
    auto fetch_operands = [&](int grp) {                       // an absent operand has a descriptor of size zero: no branches, no waits
        const __amdgpu_buffer_rsrc_t s_bias = buf(a.bias, a.bias_bytes), s_bias2 = buf(a.bias2, a.bias2_bytes),
                                     s_temb = buf(a.temb, a.temb_bytes), s_res = buf(a.res, a.res_bytes);
        const int res_compact = CONV ? 0 : a.res_compact, res_shift = res_compact == 2 ? 2 : 1;       // float rows / bf16 (16 bytes are fetched either way, 8 of them used)
#pragma unroll
        for (int it = 0; it < IPG; ++it) {
            const unsigned no = e_ok[grp * IPG + it] && !trans ? 0u : OOB, col = (unsigned)(col0 + e_c[grp * IPG + it]);
            e_bias[it] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s_bias, (col * 2u) | no, 0, 0));
            if constexpr (GEGLU) {
                e_gate[it] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s_bias, ((col + pr.N) * 2u) | no, 0, 0));
            } else {
                const unsigned r = __umul24(res_compact ? (unsigned)(m0 + e_r[grp * IPG + it]) : e_pix[grp * IPG + it], (unsigned)pr.N) + col;
                if constexpr (CONV) e_res[it].xy = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s_res, (r << 1) | no, 0, 0));
                else e_res[it] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s_res, (r << res_shift) | no, 0, 0));
                if constexpr (AM == A_MAP) {
                    e_bias2[it] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(s_bias2, (col * 2u) | no, 0, 0));
                    e_temb[it] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s_temb, ((__umul24((unsigned)e_b[grp * IPG + it], (unsigned)a.temb_stride) + col) * 4u) | no, 0, 0));
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
                        e_ss[it][v][0] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s, off, 0, 0));
                        e_ss[it][v][1] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s, off, 16, 0));
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
    // PATCH: pixel (24 bits), segment (3 bits above) of every patch row this lane loads, address in the current source; cursor: chunk, place in LDS
    unsigned px_p[PG::SLOTS], va_p[PG::SLOTS], soff_p = 0, end_p = 0, pslot = 0; int chunk_p = ch0;
    const bf16_t* ptr_p = nullptr; unsigned bytes_p = 0;
    auto set_patch_source = [&](int cc0) {
        const int i = cc0 >= a.C0 ? 1 : 0;
        ptr_p = a.src[i].p; bytes_p = a.src[i].bytes; end_p = a.src[i].pitch; soff_p = (unsigned)(cc0 - (i ? a.C0 : 0)) * 2u;
#pragma unroll
        for (int j = 0; j < PG::SLOTS; ++j) va_p[j] = (__umul24(px_p[j], end_p) + (px_p[j] >> 20 & 0x70u)) | (px_p[j] & OOB);
    };
    auto issue_patch = [&]() {                                 // SLOTS loads always
        const __amdgpu_buffer_rsrc_t rs = buf(ptr_p, chunk_p < ch1 ? bytes_p : 0u);
        unsigned char* base = ring + pslot + wave * 1024;
#pragma unroll
        for (int j = 0; j < PG::SLOTS; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(base + j * 4096), 16, va_p[j], soff_p, 0, 0);
        ++chunk_p; soff_p += 128u;
        pslot = pslot == (NPB - 1) * PG::BYTES ? 0u : pslot + PG::BYTES;
        if (soff_p == end_p && chunk_p < ch1) set_patch_source(a.C0);
    };
    if constexpr (PATCH) {
        // lane's patch rows: strip, row and column in the ringed strip; the strip's first output pixel is known to the lane of its row
#pragma unroll
        for (int j = 0; j < PG::SLOTS; ++j) {
            const int p = j * 32 + lrow, strip = p / PG::PIX, q = p - strip * PG::PIX, r0 = strip * (PG::H * PATCH);
            const int iy = __shfl(ry, r0 & (BM - 1)) - 1 + q / (PATCH + 2), ix = __shfl(rx, r0 & (BM - 1)) - 1 + q % (PATCH + 2), b = __shfl((int)rb, r0 & (BM - 1));
            const bool in = strip < PG::STRIPS && m0 + r0 < rows && (unsigned)iy < (unsigned)a.Hin && (unsigned)ix < (unsigned)a.Win;
            const unsigned pix = __umul24(__umul24((unsigned)b, (unsigned)a.Hin) + iy, (unsigned)a.Win) + ix;
            px_p[j] = in ? pix | (unsigned)((lane & 7) ^ PG::swizzle(p)) << 24 : OOB;
        }
        set_patch_source(ch0 * 64);
        if (nside > 0) {
            const unsigned o0 = my_row < rows ? rpix : OOB;
#pragma unroll
            for (int l = 0; l < TM; ++l) out_s[l] = (unsigned)__shfl((int)o0, l * 32 + lrow);
            const unsigned pitch2 = (unsigned)a.K2 * 2u;
#pragma unroll
            for (int l = 0; l < BL; ++l) vb_s[l] = __umul24((unsigned)(by * BN + l * 32 + lrow), pitch2) + seg0;
            soff_w2 = (unsigned)sd0 * 128u;
            set_side(sd0 * 64);
        }
#pragma unroll
        for (int s = FIRST_A; s < 0; ++s) {
            if (s % 3 == 0) issue_patch();
            if (s >= -WAHEAD) issue_step();
        }
    } else if constexpr (AM == A_MAP) {
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
    if constexpr (!PATCH)
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
    if constexpr (PATCH) {
        // Every wave multiplies its 16-deep slice of 64 channels over the whole tile.  Behind each product of step s its registers
        // take the operands of step s + 1, which have landed in LDS for all waves (the barrier says so); that barrier
        // also says that every wave is done with what step s - 1 read, which is refilled.
        const int slice = wave * 2 + (lane >> 5);
        unsigned rp[9][TM];                             // operand A under each tap: place in a patch
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int r = i * 32 + (lane & 31), q = r / (PG::H * PATCH) * PG::PIX + r % (PG::H * PATCH) / PATCH * (PATCH + 2) + r % PATCH;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int p = q + t / 3 * (PATCH + 2) + t % 3;
                rp[t][i] = (unsigned)(p * 128 + ((slice ^ PG::swizzle(p)) * 16));
            }
        }
        bf16x8_t fa[3][TM], fb[3][TN];
        auto read_b = [&](bf16x8_t (&f)[TN], unsigned slot, int row) {
#pragma unroll
            for (int n = 0; n < TN; ++n) f[n] = *reinterpret_cast<const bf16x8_t*>(wring + slot + rd_own + (row + n * 32) * 128);
        };
        auto read_a = [&](bf16x8_t (&f)[TM], unsigned patch, int tap) {
#pragma unroll
            for (int i = 0; i < TM; ++i) f[i] = *reinterpret_cast<const bf16x8_t*>(ring + patch + rp[tap][i]);
        };
        auto multiply = [&](const bf16x8_t (&x)[TM], const bf16x8_t (&w)[TN]) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int n = 0; n < TN; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n], x[i], acc[i][n], 0, 0, 0);
        };
        auto next_slot = [&](unsigned s) { return s == (NB - 1) * WSTAGE ? 0u : s + WSTAGE; };
        unsigned rslot = 0, rpatch = 0;                 // where the step whose operands are read next lies
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(patch_flight0(WAHEAD, NPB, LB, PG::SLOTS)) : "memory");
#pragma unroll
        for (int j = 0; j < 3; ++j) { read_a(fa[j], 0, j); read_b(fb[j], 0, j * BN); }
#pragma unroll 1
        for (int c = ch0; c < ch1; ++c) {
            auto step = [&](auto ky_) {
                constexpr int ky = decltype(ky_)::value, after = (ky + 1) % 3;
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(patch_flight(ky, WAHEAD, NPB, LB, PG::SLOTS)) : "memory");
                if (ky == 2) rpatch = rpatch == (NPB - 1) * PG::BYTES ? 0u : rpatch + PG::BYTES;
                rslot = next_slot(rslot);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    multiply(fa[j], fb[j]);
                    read_a(fa[j], rpatch, after * 3 + j); read_b(fb[j], rslot, j * BN);     // behind the last chunk: not used
                    __builtin_amdgcn_sched_barrier(0);
                    if (j == 0) {
                        if (ky == 0) issue_patch();
                        issue_step();
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{}); step(std::integral_constant<int, 2>{});
        }
        // side product: a ring slot holds BM rows of A, then BN rows of W
        if (nside > 0) {
            auto read_side = [&]() {
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[0][i] = *reinterpret_cast<const bf16x8_t*>(wring + rslot + rd_own + i * 4096);
                read_b(fb[0], rslot, BM);
            };
            read_side();
#pragma unroll 1
            for (int e = 0; e < nside; ++e) {
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((WAHEAD - 2) * LB) : "memory");
                rslot = next_slot(rslot);
                multiply(fa[0], fb[0]);
                read_side();
                __builtin_amdgcn_sched_barrier(0);
                issue_step();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else if constexpr (SHARED) {
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
    f32x4_t v[ITEMS], g[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) v[it] = g[it] = f32x4_t{0.f, 0.f, 0.f, 0.f};
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
                    *reinterpret_cast<f32x4_t*>(&part[(wave * GROWS + i * 32 + (lane & 31)) * PITCH + j * 32 + q * 8 + (lane >> 5) * 4]) =
                        f32x4_t{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                }
        __syncthreads();
        if (trans) {
#pragma unroll
            for (int it = grp * IPG; it < (grp + 1) * IPG; ++it)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float* p = &part[(w * GROWS + e_r[it] - grp * GROWS) * PITCH + e_c[it]];
                    v[it] += f32x4_t{p[0], p[PITCH], p[2 * PITCH], p[3 * PITCH]};
                }
        } else {
#pragma unroll
            for (int it = grp * IPG; it < (grp + 1) * IPG; ++it)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float* p = &part[(w * GROWS + e_r[it] - grp * GROWS) * PITCH + e_c[it]];
                    v[it] += *reinterpret_cast<const f32x4_t*>(p);
                    if (GEGLU) g[it] += *reinterpret_cast<const f32x4_t*>(p + OW);
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
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v[it]), s_part, off, 0, 17);
            if (GEGLU) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, g[it]), s_part, off + BM * OW * 4, 0, 17);
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
        for (int it = 0; it < ITEMS; ++it) v[it] = g[it] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int z = 0; z < a.splits; ++z) {            // split order, whoever is last
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const unsigned off = (base + z) * SLOT + (unsigned)(it * NT + tid) * 16u;
                v[it] += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s_part, off, 0, 17));
                if (GEGLU) g[it] += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s_part, off + BM * OW * 4, 0, 17));
            }
        }
    }

    // ---- epilogue: sum, biases, gate, then time projection + residual as one term; stores
    bf16_t* const outp = sect == 0 ? pr.out0 : sect == 1 ? a.out[1] : a.out[2];
    const int scol0 = col0 - sect * pr.sect_n;
    if constexpr (CONV) {
        // A group's results are packed in registers, the next group's operands requested, and only then stored: behind the
        // stores the loads would wait for them.
#pragma unroll
        for (int grp = 0; grp < GROUPS; ++grp) {
            u32x2_t y[IPG], yv[IPG][2];
#pragma unroll
            for (int it = 0; it < IPG; ++it) {
                const f32x4_t sum = v[grp * IPG + it];
                float x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    auto part = [q](const u32x2_t& w) { return q & 1 ? hi16(w[q >> 1]) : lo16(w[q >> 1]); };
                    const float res = part(u32x2_t{e_res[it][0], e_res[it][1]});
                    x[q] = sum[q] + part(e_bias[it]);
                    x[q] += part(e_bias2[it]);
                    x[q] += res + __uint_as_float(e_temb[it][q]);
                }
                y[it] = u32x2_t{f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (i < a.nview) {                  // as put_views4
                        float u[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const u32x4_t& ss = e_ss[it][i][q >> 1];
                            u[q] = view_scale(q & 1 ? hi16(y[it][q >> 1]) : lo16(y[it][q >> 1]), __uint_as_float(ss[(q & 1) * 2]), __uint_as_float(ss[(q & 1) * 2 + 1]));
                        }
                        if (a.view[i].silu) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) u[q] = silu_f(u[q]);
                        }
                        yv[it][i] = u32x2_t{f2bf2(u[0], u[1]), f2bf2(u[2], u[3])};
                    }
            }
            if (grp + 1 < GROUPS) fetch_operands(grp + 1);
#pragma unroll
            for (int it = 0; it < IPG; ++it) {
                const int e = grp * IPG + it;
                if (!e_ok[e]) continue;
                *(FISE_AS1 u32x2_t*)(outp + (size_t)e_pix[e] * pr.N + col0 + e_c[e]) = y[it];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (i < a.nview) *(FISE_AS1 u32x2_t*)(a.view[i].dst + (size_t)e_pix[e] * a.view[i].dstC + a.view[i].c_off + col0 + e_c[e]) = yv[it][i];
            }
        }
        return;
    }
    if (trans) {
        const unsigned HW = (unsigned)(a.Ho * a.Wo);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (!e_ok[it]) continue;
            FISE_AS1 bf16_t* q = (FISE_AS1 bf16_t*)(outp + ((size_t)e_b[it] * pr.sect_n + scol0 + e_c[it]) * HW + (e_pix[it] - (unsigned)e_b[it] * HW));
            *(FISE_AS1 u32x2_t*)q = u32x2_t{f2bf2(v[it][0], v[it][1]), f2bf2(v[it][2], v[it][3])};
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
            const u32x4_t w = e_res[gi];
            f32x4_t r = a.res_compact == 2 ? __builtin_bit_cast(f32x4_t, w) : f32x4_t{lo16(w[0]), hi16(w[0]), lo16(w[1]), hi16(w[1])};
            if constexpr (AM == A_MAP) {
                x[0] += lo16(e_bias2[gi][0]); x[1] += hi16(e_bias2[gi][0]); x[2] += lo16(e_bias2[gi][1]); x[3] += hi16(e_bias2[gi][1]);
                r += __builtin_bit_cast(f32x4_t, e_temb[gi]);
            }
            x[0] += r[0]; x[1] += r[1]; x[2] += r[2]; x[3] += r[3];
        }
        if (!e_ok[it]) continue;
        const int scol = scol0 + e_c[it];
        const size_t gm = (size_t)(m0 + e_r[it]);
        if (omode == OUT_TOKENS_T) {
            const size_t HW = (size_t)a.Ho * a.Wo;
            FISE_AS1 bf16_t* q = (FISE_AS1 bf16_t*)(outp + ((size_t)e_b[it] * pr.sect_n + scol) * HW + (e_pix[it] - (unsigned)e_b[it] * (unsigned)HW));
#pragma unroll
            for (int t = 0; t < 4; ++t) q[t * HW] = f2bf(x[t]);
            continue;
        }
        const u32x2_t packed = {f2bf2(x[0], x[1]), f2bf2(x[2], x[3])};
        if (omode == OUT_COMPACT_F32) {
            if (outp) *(FISE_AS1 f32x4_t*)(reinterpret_cast<float*>(outp) + gm * pr.sect_n + scol) = f32x4_t{x[0], x[1], x[2], x[3]};
            if (a.mirror) *(FISE_AS1 u32x2_t*)(a.mirror + gm * pr.sect_n + scol) = packed;
        } else if (omode == OUT_COMPACT) {
            *(FISE_AS1 u32x2_t*)(outp + gm * pr.sect_n + scol) = packed;
        } else {
            *(FISE_AS1 u32x2_t*)(outp + (size_t)e_pix[it] * pr.sect_n + scol) = packed;
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

// Place of this workgroup in the order in which its XCD should work: consecutive workgroups go round-robin to the 8 XCDs; every XCD
// gets a contiguous run of (bz, by, bx), bx fastest, so that a slice of the weights is pulled into one L2.
__device__ __forceinline__ int xcd_order(int total) {
    const int w = blockIdx.x, chunk = total >> 3;
    return w < (chunk << 3) ? (w & 7) * chunk + (w >> 3) : w;
}

template <int TM, int TN, int NW, int NST, int AM, bool GEGLU, bool SHARED, int PATCH = 0, int NPB = 0>
__global__ __launch_bounds__(64 * NW, SHARED && TN == 2 && !PATCH ? 3 : 1) void wave_gemm_kernel(const IgemmArgs a) {
    asm volatile("" ::"s"(a.gx), "s"(a.gy), "s"(a.splits), "s"(a.d_gx.mul), "s"(a.d_gy.mul));
    const int w = xcd_order(a.gx * a.gy * a.splits);
    const unsigned t = fdiv((unsigned)w, a.d_gx);
    const int bz = (int)fdiv(t, a.d_gy);
    wave_gemm_tile<TM, TN, NW, NST, AM, GEGLU, SHARED, PATCH, NPB>(a, Product{a.w, a.N, a.sect_n, a.out[0], a.out_mode[0]}, w - (int)t * a.gx, (int)t - bz * a.gy, bz);
}

// Several products of the same compact rows, each with weights, width and destination of its own, as one launch.
template <int TM, int TN, int NW, int NST, bool SHARED>
__global__ __launch_bounds__(64 * NW, SHARED ? 3 : 1) void wave_gemm_group_kernel(const IgemmArgs a, const GemmGroup grp) {
    const int w = xcd_order(a.gx * a.gy);
    const int t = (int)fdiv((unsigned)w, a.d_gx);
    int g = 0;
#pragma unroll
    for (int i = 1; i < GEMM_GROUP; ++i) g += t >= grp.first[i];        // column tiles of all products, one behind the other
    wave_gemm_tile<TM, TN, NW, NST, A_ROWS, false, SHARED>(a, Product{grp.w[g], grp.N[g], grp.N[g], grp.out[g], grp.mode[g]}, w - t * a.gx, t - grp.first[g], 0);
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

template <int TM, int TN, int NST, int AM, bool GEGLU, bool SHARED = false, int PATCH = 0, int NPB = 0>
static int launch_tile(const IgemmArgs& a, hipStream_t st) {
    constexpr int NW = 4, lds = PATCH ? NPB * Patch<32 * TM, PATCH ? PATCH : 8>::BYTES + NST * 3 * 32 * TN * 128 : (SHARED ? 1 : NW) * NST * (32 * TM + 32 * TN) * 128;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    // raised once per instantiation (initialisation of a function-local static is thread safe)
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wave_gemm_kernel<TM, TN, NW, NST, AM, GEGLU, SHARED, PATCH, NPB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "wave gemm: cannot raise the dynamic LDS limit");
    const double rows = (double)a.B * a.Ma, ncols = a.geglu ? 2.0 * a.N : a.N, K = (double)a.K + a.K2;
    {
        ProfileScope prof(GEGLU ? PROF_IGEMM_GEGLU : AM == A_MAP ? PROF_IGEMM : PROF_ROWS_GEMM, 2.0 * rows * ncols * K, 2.0 * (ncols * K + rows * (a.C0 + a.C1 + a.S0 + a.S1) + rows * a.N), st);
        hipLaunchKernelGGL((wave_gemm_kernel<TM, TN, NW, NST, AM, GEGLU, SHARED, PATCH, NPB>), dim3((unsigned)(a.gx * a.gy * a.splits)), dim3(64 * NW), lds, st, a);
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

// Compact rows of one section from here on: linear_wide.hip (float rows) and igemm.hip's 64 x 128 and 64 x 64 tiles (8192 x 320 x 320 12.8 against 14.3 us,
// 2048 x 640 x 640 12.7 against 13.3 us on shared tiles).
constexpr int BLOCK_ROWS = 2048;
bool wave_gemm_takes(const IgemmArgs& a) {
    return wave_gemm_fits(a) && (a.B * a.Ma < BLOCK_ROWS || !a.a_compact || a.geglu || a.nsect > 1);
}

// 3x3 products over pixels of square tiles whose strips have a patch form, into one map (wider tiles, rectangles, stride 2 and upsampling
// keep the forms that gather a tap at a time).
static bool patch_fits(const IgemmArgs& a) {
    return !a.a_compact && a.ksize == 3 && a.stride == 1 && !a.ups && (a.tile_w == 0 || a.tile_w == a.tile) && (a.tile == 2 || a.tile == 4 || a.tile == 8) &&
           a.nsect == 1 && a.out_mode[0] == OUT_MAP && !(a.res && a.res_compact);
}

static TileChoice choose_tile(const IgemmArgs& a, const IgemmWorkspace* ws) {
    GemmShape g;
    g.rows = a.B * a.Ma; g.N = a.N; g.K = a.K; g.K2 = a.K2; g.tile = a.tile; g.geglu = a.geglu; g.patches = patch_fits(a);
    g.one_map = !a.a_compact && a.nsect == 1 && a.out_mode[0] == OUT_MAP && !(a.res && a.res_compact);
    return choose_tile(g, ws && ws->counters && ws->partial ? ws->partial_bytes : 0);
}

// Stages in LDS: as many as it holds (a chunk's weights for a column tile of 32 are 36 KB, its patch 8 - 32 KB).
template <int T>
static int launch_patches(const IgemmArgs& a, int tm, int tn, hipStream_t st) {
    if constexpr (T > 2)
        if (tm == 1) return launch_tile<1, 1, 9, A_MAP, false, true, T, 3>(a, st);
    if (tn == 1) return launch_tile<2, 1, T == 8 ? 9 : T == 4 ? 8 : 5, A_MAP, false, true, T, 3>(a, st);
    return launch_tile<2, 2, T == 8 ? 5 : 4, A_MAP, false, true, T, 2>(a, st);
}

// The products of a group as one launch (no K split).  One by one they are a few dozen workgroups each that wait for one another's
// launch: queries, keys and values of 640 rows of 320 channels three launches of 4.7 -> one of 6.  Many columns (keys and values of a prompt for all
// blocks) belong to rows_group.hip.
template <int TM, int TN, int NST, bool SHARED>
static int launch_group_tile(const IgemmArgs& a, const GemmGroup& g, hipStream_t st) {
    constexpr int NW = 4, lds = (SHARED ? 1 : NW) * NST * (32 * TM + 32 * TN) * 128;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&wave_gemm_group_kernel<TM, TN, NW, NST, SHARED>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "wave gemm group: cannot raise the dynamic LDS limit");
    {
        const double rows = (double)a.B * a.Ma;
        ProfileScope prof(PROF_ROWS_GEMM, 2.0 * rows * a.N * a.K, 2.0 * ((double)a.N * a.K + rows * a.K + rows * a.N), st);
        hipLaunchKernelGGL((wave_gemm_group_kernel<TM, TN, NW, NST, SHARED>), dim3((unsigned)(a.gx * a.gy)), dim3(64 * NW), lds, st, a, g);
    }
    FISE_CHECK_LAUNCH("wave gemm group");
    return FISE_OK;
}

int launch_igemm_group(const IgemmArgs& base, const GemmProduct* p, int n, hipStream_t st) {
    IgemmArgs a = base;
    a.nsect = 1; a.sect_n = a.N; a.splits = 1;
    bool grouped = n > 1 && n <= GEMM_GROUP && !a.bias && !a.temb && !a.res && !a.nview && !a.geglu && !a.ln_out && a.a_compact && a.C0 == a.K;
    int cols = 0; bool pix = false, tokens = false;
    for (int i = 0; i < n; ++i) {
        IgemmArgs b = a;
        b.N = b.sect_n = p[i].N;
        grouped &= wave_gemm_fits(b) && p[i].N % 64 == 0;
        cols += p[i].N; pix |= p[i].mode != OUT_COMPACT; tokens |= p[i].mode == OUT_TOKENS_T;
    }
    if (!grouped || a.B * a.Ma <= 0) {                  // one by one
        for (int i = 0; i < n; ++i) {
            a.w = p[i].w; a.N = a.sect_n = p[i].N; a.out[0] = p[i].out; a.out_mode[0] = p[i].mode;
            if (int e = launch_igemm(a, nullptr, st)) return e;
        }
        return FISE_OK;
    }
    if (rows_group_takes(a, p, n)) return launch_rows_group(a, p, n, st);
    a.N = cols;
    const TileChoice c = choose_tile(a, nullptr);
    GemmGroup g{};
    int tiles = 0;
    for (int i = 0; i < GEMM_GROUP; ++i) {
        g.first[i] = i < n ? tiles : 1 << 30;
        if (i >= n) continue;
        g.w[i] = p[i].w; g.out[i] = p[i].out; g.N[i] = p[i].N; g.mode[i] = p[i].mode;
        tiles += p[i].N / (32 * c.tn);
    }
    a.out_mode[0] = tokens ? OUT_TOKENS_T : pix ? OUT_MAP : OUT_COMPACT;
    a.gx = ceil_div(a.B * a.Ma, 32 * c.tm); a.gy = tiles; a.kper = a.K / 64;
    prepare(a, a.N);
    if (c.kind == SHARED_RING) return launch_group_tile<2, 2, 3, true>(a, g, st);
    if (c.tm == 2) return launch_group_tile<2, 2, 2, false>(a, g, st);
    return c.tn == 2 ? launch_group_tile<1, 2, 2, false>(a, g, st) : launch_group_tile<1, 1, 2, false>(a, g, st);
}

int launch_wave_gemm(IgemmArgs a, const IgemmWorkspace* ws, hipStream_t st) {
    const int rows = a.B * a.Ma, ncols = a.geglu ? 2 * a.N : a.N, nsteps = (a.K + a.K2) / 64;
    const TileChoice c = choose_tile(a, ws);
    a.splits = c.splits;
    if (c.kind == PATCHES) { a.kper = ceil_div(a.K / 576, c.splits); a.kper2 = ceil_div(a.K2 / 64, c.splits); }
    else a.kper = ceil_div(nsteps, c.splits);
    a.gx = ceil_div(rows, 32 * c.tm); a.gy = c.kind == WIDE ? a.N / 80 : ceil_div(ncols, 32 * c.tn);
    prepare(a, ncols);
    // 384 x 640 x 11520 in 12 row tiles: 21.9 -> 18.4 us, 512 x 1280 x 11520 in eight 38.9 -> 34.9; three row tiles, which have four times
    // the lines each, 26.1 -> 28.4
    a.touch = a.gx >= 8;
    if (a.splits > 1) {
        a.partial = ws->partial; a.counters = ws->counters;
        if (!ws->counters_zeroed) {                     // once per call: every launch leaves its counters at zero
            hipLaunchKernelGGL(zero_ints_kernel, dim3(ceil_div(IGEMM_COUNTERS, 256)), dim3(256), 0, st, ws->counters, IGEMM_COUNTERS);
            FISE_CHECK_LAUNCH("zero counters");
            ws->counters_zeroed = true;
        }
    }
    int e;
    if (c.kind == PATCHES) e = a.tile == 8 ? launch_patches<8>(a, c.tm, c.tn, st) : a.tile == 4 ? launch_patches<4>(a, c.tm, c.tn, st) : launch_patches<2>(a, c.tm, c.tn, st);
    else if (c.kind == WIDE) e = launch_conv_patch(a, c.tm, st);
    else if (c.kind == BLOCK) e = launch_tile<2, 5, 4, A_MAP, false, true>(a, st);
    else if (c.kind == SHARED_RING)
        e = a.geglu ? launch_tile<2, 2, 3, A_ROWS, true, true>(a, st) : a.a_compact ? launch_tile<2, 2, 3, A_ROWS, false, true>(a, st) : launch_tile<2, 2, 3, A_MAP, false, true>(a, st);
    else if (a.geglu) e = c.tm == 1 ? launch_tile<1, 2, 2, A_ROWS, true>(a, st) : launch_tile<2, 2, 2, A_ROWS, true>(a, st);
    else if (a.a_compact)
        e = c.tm == 2 ? launch_tile<2, 2, 2, A_ROWS, false>(a, st) : c.tn == 2 ? launch_tile<1, 2, 2, A_ROWS, false>(a, st) : launch_tile<1, 1, 2, A_ROWS, false>(a, st);
    else
        e = c.tm == 2 ? launch_tile<2, 2, 2, A_MAP, false>(a, st) : c.tn == 2 ? launch_tile<1, 2, 2, A_MAP, false>(a, st) : launch_tile<1, 1, 2, A_MAP, false>(a, st);
    if (e) return e;
    if (a.ln_out) {
        if (a.nsect != 1 || a.out_mode[0] != OUT_COMPACT_F32 || a.geglu || !a.ln_gamma || !a.ln_beta)
            return fail(FISE_ERR_SHAPE, "igemm: LayerNorm output needs one float compact section");
        return launch_ln_rows(a.out[0], 1, rows, a.N, a.ln_gamma, a.ln_beta, a.ln_eps, a.ln_out, nullptr, 1, 1, 1, 1, 1, st);
    }
    return FISE_OK;
}

}  // namespace fise
