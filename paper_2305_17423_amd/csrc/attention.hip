// Active-query attention on bf16 MFMA: each wave owns 32 gathered queries of one
// (batch, head) and streams keys in blocks of 64 through LDS with an online
// softmax.  Scores are computed transposed (S^T = K Q^T) so that a lane keeps one
// query's running max / sum to itself, and the output is accumulated transposed
// (O^T = V^T P^T), which is why V operands are stored keys-innermost.
//
// With few active queries there are few (query tile, head, batch) workgroups, so
// the key range is also split over workgroups: each writes an unnormalised partial
// (running max, sum, output) and a second small kernel merges the partials in
// split order.  The next key block is fetched into registers while the current
// one is being multiplied; the LDS hand-over uses a barrier that does not wait for
// those loads.
#include <algorithm>
#include <type_traits>
#include "attention_choice.h"
#include "attention_keys.h"
#include "igemm.h"
#include "profile.h"

namespace fise {

constexpr int AT_QW = 32;         // queries per wave
static_assert(AT_BQ == 4 * AT_QW, "four waves");

__device__ __forceinline__ void at_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A query's two lanes: the swap leaves the lower half's value in one result and the upper half's in the other.  An instruction where a shuffle
// is a trip to the LDS between the scores and their exponentials (and the sums meet once, behind the last block): 2 x 9216 queries and keys of
// 8 x 40 channels 436 -> 421 us, 2 x 4096 of 8 x 160 216 -> 212, 2 x 1024 of 8 x 160 37.8 -> 35.9, 2 x 768 x 4096 keys of 8 x 40 unchanged.
__device__ __forceinline__ float2 at_halves(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return make_float2(__uint_as_float(p[0]), __uint_as_float(p[1]));
#else
    return make_float2(x, x);
#endif
}

// Workgroup -> (query tile qt, head h, batch element b, key split sp).  The grid is one-dimensional
// and consecutive workgroups go round-robin to the 8 XCDs (one L2 each): workgroup w takes position
// (w % 8) * (total / 8) + w / 8 of the (b, sp, h, qt) order, qt fastest, so the query tiles that
// stream the same K / V slice run on one XCD and the slice is fetched from HBM once, not eight times.
struct AtPlace { int qt, h, b, sp; };
__device__ __forceinline__ AtPlace at_place(int nqt, int heads, int B, int splits, FastDiv d_nqt, FastDiv d_heads, FastDiv d_splits) {
    const int total = nqt * heads * B * splits, chunk = total >> 3;
    int w = blockIdx.x;
    if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
    const int t = (int)fdiv(w, d_nqt), u = (int)fdiv(t, d_heads), b = (int)fdiv(u, d_splits);
    return {w - t * nqt, t - u * heads, b, u - b * splits};
}

// What both kernels of many queries begin and end with.  Query fragments: B operand of S^T = K Q^T (column = query, 8 consecutive head-dim elements)
template <int KD> __device__ __forceinline__ void at_queries(bf16x8_t (&qf)[KD], const bf16_t* __restrict__ q, int M, int C, int b, int h, int qrow, bool qok, int hl, int d) {
#pragma unroll
    for (int ks = 0; ks < KD; ++ks) {
        const int c = ks * 16 + hl * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (qok && c < d) v = *reinterpret_cast<const uint4*>(q + ((size_t)b * M + qrow) * C + h * d + c);
        qf[ks] = *reinterpret_cast<bf16x8_t*>(&v);
    }
}
// Store: lane holds query l32, head-dim rows i*32 + (e/4)*8 + hl*4 + e%4: four consecutive elements of e are
// four consecutive channels (d is a multiple of 8, so a group of four is inside the head or outside it as a whole)
template <int DB> __device__ __forceinline__ void at_store(const f32x16_t (&oacc)[DB], float m_run, float l_run, bool qok, int splits, int B, int M, int C, int heads, int b, int h, int sp,
                                                           int qrow, int hl, int d, bf16_t* __restrict__ out, float* __restrict__ part_o, float* __restrict__ part_ml) {
    const float2 lh = at_halves(l_run);
    l_run = lh.x + lh.y;
    if (!qok) return;
    if (splits == 1) {
        const float inv = 1.0f / l_run;
        bf16_t* o = out + ((size_t)b * M + qrow) * C + h * d;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int r = i * 32 + q4 * 8 + hl * 4;
                if (r < d)
                    *reinterpret_cast<uint2*>(o + r) = make_uint2(f2bf2(oacc[i][4 * q4] * inv, oacc[i][4 * q4 + 1] * inv),
                                                                  f2bf2(oacc[i][4 * q4 + 2] * inv, oacc[i][4 * q4 + 3] * inv));
            }
    } else {
        // unnormalised partial of this key range: O[sp][b][qrow][h*d + r], (m, l)[sp][b][h][qrow]
        float* po = part_o + (((size_t)sp * B + b) * M + qrow) * C + h * d;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int r = i * 32 + q4 * 8 + hl * 4;
                if (r < d)
                    *reinterpret_cast<float4*>(po + r) = make_float4(oacc[i][4 * q4], oacc[i][4 * q4 + 1], oacc[i][4 * q4 + 2], oacc[i][4 * q4 + 3]);
            }
        if (hl == 0) {
            float* pm = part_ml + ((((size_t)sp * B + b) * heads + h) * M + qrow) * 2;
            pm[0] = m_run; pm[1] = l_run;
        }
    }
}

// KD: 16-wide steps over the head dim; DB: 32-row blocks of the output head dim; EXACT: the head dim is 16 KD (80, 160: the set-up
// of a short launch is instructions, and most of its conditions and address terms are constants then).
// What bounds it: few queries, the round trips of the key blocks (~0.9 us each with two blocks in flight, heads up to 96; ~2 us
// with one); many queries, the exponentials and the other ~100 vector instructions per 64 keys.  The wide heads sit right below
// 256 registers, where a CU still holds two workgroups: 2 x 4096 queries and keys of 8 x 160 channels 212 us, at 262
// registers half as fast again (325 when it was 226).
template <int KD, int DB, bool EXACT>
__global__ __launch_bounds__(256, 2) void attention_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ K,
                                                           const bf16_t* __restrict__ Vt, int B, int M, int n_keys, int n_stride,
                                                           int C, int d_arg, float scale_log2e, int splits, int nqt, int heads,
                                                           FastDiv d_nqt, FastDiv d_heads, FastDiv d_splits, int chunk_mul,
                                                           bf16_t* __restrict__ out, float* __restrict__ part_o, float* __restrict__ part_ml) {
    constexpr int DP = KD * 16;
    constexpr int KP = DP + 8;            // K tile pitch (bf16)
    constexpr int VP = AT_BKV + 8;        // V^T tile pitch
    constexpr int KCH = AT_BKV * (DP / 8);        // 16-byte chunks of the K tile
    constexpr int VCH = DB * 32 * (AT_BKV / 8);   // and of the V^T tile
    constexpr int KL = (KCH + 255) / 256, VL = (VCH + 255) / 256;
    __shared__ __attribute__((aligned(16))) bf16_t Ks[AT_BKV][KP];
    __shared__ __attribute__((aligned(16))) bf16_t Vs[DB * 32][VP];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hl = lane >> 5, l32 = lane & 31;
    const auto [qt, h, b, sp] = at_place(nqt, heads, B, splits, d_nqt, d_heads, d_splits);
    const int qrow = qt * AT_BQ + wave * AT_QW + l32;
    const bool qok = qrow < M;
    const int d = EXACT ? DP : d_arg, dchunks = d / 8;

    // key blocks of this split
    const int nblocks = (n_keys + AT_BKV - 1) / AT_BKV;
    const int per = (nblocks + splits - 1) / splits;
    const int blk0 = sp * per, blk1 = min(nblocks, blk0 + per);

    bf16x8_t qf[KD];
    at_queries(qf, q, M, C, b, h, qrow, qok, hl, d);

    f32x16_t oacc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;                // l: of this lane's half of the keys until the end

    // ---- register staging of key blocks.  Thread slot j covers chunk e = tid + 256 j of the block's real data:
    // K rows of d / 8 chunks (key e / dchunks, chunk e % dchunks), V^T rows of 8 chunks (row e / 8 < d, keys
    // (e % 8) * 8 ..).  Everything that depends only on the slot is worked out once; a block costs one pointer
    // bump and one load per slot.  The head-dim columns of the K tile past d are zeroed once and never written
    // again (V^T rows past d only reach output rows that are not stored).  Keys that do not exist can only occur in the
    // last block of the whole range, which may be the first: its loads go to the last key, or chunk of eight, that exists
    // (attention_keys.h; all of them unconditional: behind a branch each, they were a round trip each) and what
    // they bring is replaced by zeros on the way into the LDS tiles.
    constexpr int PFD = (KL + VL <= 6) ? 2 : 1;       // key blocks in flight (small heads can afford two in registers)
    uint4 rk[PFD][KL], rv[PFD][VL];
    const bf16_t* pk[KL]; const bf16_t* pv[VL];        // source of the slot in key block 0
    int kkey[KL];                                      // key of the K slot within a block (-1: slot unused)
    const int vkey = (tid & 7) * 8;                    // first key of the V^T slots (256 threads: whole rows of 8 chunks)
    bf16_t* sk[KL]; bf16_t* sv[VL];                    // destination in the LDS tiles
    auto v_used = [&](int j) { return (EXACT && VCH == 256 * VL && DB * 32 == DP) || ((tid + 256 * j) >> 3) < d; };
#pragma unroll
    for (int j = 0; j < KL; ++j) {
        const int e = tid + 256 * j;
        const int kk = EXACT ? e / (DP / 8) : (e * chunk_mul) >> 16, c8 = e - kk * dchunks;      // e / dchunks: e < 1280, dchunks <= 20
        const bool used = (EXACT && KCH == 256 * KL) || e < AT_BKV * dchunks;
        kkey[j] = used ? kk : -1;
        pk[j] = K + (used ? ((size_t)b * n_keys + kk) * C + h * d + c8 * 8 : 0);
        sk[j] = &Ks[used ? kk : 0][used ? c8 * 8 : 0];
    }
#pragma unroll
    for (int j = 0; j < VL; ++j) {                     // (unused: the chunk of the same keys in the first row)
        const int r = (tid + 256 * j) >> 3;
        pv[j] = Vt + (v_used(j) ? ((size_t)b * C + h * d + r) * n_stride : 0) + vkey;
        sv[j] = &Vs[v_used(j) ? r : 0][vkey];
    }
    for (int e = tid; e < AT_BKV * (DP / 8 - dchunks); e += 256) *reinterpret_cast<uint4*>(&Ks[e % AT_BKV][d + e / AT_BKV * 8]) = make_uint4(0, 0, 0, 0);
    auto fetch = [&](int blk, int slot) {
        const int k0 = blk * AT_BKV;
        if (k0 + AT_BKV <= n_keys) {                     // uniform: a block of existing keys
#pragma unroll
            for (int j = 0; j < KL; ++j) rk[slot][j] = *reinterpret_cast<const uint4*>(pk[j] + (size_t)k0 * C);
#pragma unroll
            for (int j = 0; j < VL; ++j) rv[slot][j] = *reinterpret_cast<const uint4*>(pv[j] + k0);
        } else {
            const int last = n_keys - 1 - k0;            // last key of the block
#pragma unroll
            for (int j = 0; j < KL; ++j) rk[slot][j] = *reinterpret_cast<const uint4*>(pk[j] + (long long)at_key_shift(k0, last, kkey[j]) * C);
#pragma unroll
            for (int j = 0; j < VL; ++j) rv[slot][j] = *reinterpret_cast<const uint4*>(pv[j] + at_value_shift(k0, last, vkey));
            // keeps the loads of the two branches apart: merged, every whole block pays for selecting its shifts (2 x 4096
            // queries and keys of 8 x 160 channels 229 -> 226 us, 2 x 192 queries 256 keys 14.2 -> 13.5)
            asm volatile("");
        }
    };
    auto stash = [&](int blk, int slot) {
        const int nk = n_keys - blk * AT_BKV;            // keys of this block that exist
        if (__builtin_amdgcn_readfirstlane(nk < AT_BKV)) {
#pragma unroll
            for (int j = 0; j < KL; ++j)
                if (kkey[j] >= nk) rk[slot][j] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < VL; ++j) {
                const int nv = nk - vkey;             // keys of this chunk that exist
                auto keep = [&](unsigned w, int t) { return nv > t + 1 ? w : nv > t ? w & 0xffffu : 0u; };
                const uint4 v = rv[slot][j];
                rv[slot][j] = make_uint4(keep(v.x, 0), keep(v.y, 2), keep(v.z, 4), keep(v.w, 6));
            }
        }
#pragma unroll
        for (int j = 0; j < KL; ++j)
            if (kkey[j] >= 0) *reinterpret_cast<uint4*>(sk[j]) = rk[slot][j];
#pragma unroll
        for (int j = 0; j < VL; ++j)
            if (v_used(j)) *reinterpret_cast<uint4*>(sv[j]) = rv[slot][j];
    };

    if (blk0 < blk1) {
#pragma unroll
        for (int s = 0; s < PFD; ++s) fetch(min(blk0 + s, blk1 - 1), s);
    }
    // The query fragments must have ARRIVED before the key loop is entered: while their loads are still counted as
    // outstanding at the loop head, the compiler's wait-count bookkeeping (merged over the loop's paths) puts a
    // wait for ALL loads in front of the first MFMA of every iteration, i.e. right behind the prefetch of the next
    // key block, which then never overlaps anything.  Naming the fragments as operands here, behind the first key blocks' loads, places that wait once.
#pragma unroll
    for (int ks = 0; ks < KD; ++ks) asm volatile("" ::"v"(qf[ks]));
    for (int blk0u = blk0; blk0u < blk1; blk0u += PFD) {
#pragma unroll
      for (int slot = 0; slot < PFD; ++slot) {
        const int blk = blk0u + slot;
        if (blk >= blk1) break;                            // uniform across the workgroup
        const int k0 = blk * AT_BKV;
        at_lds_barrier();                                  // previous block fully consumed
        stash(blk, slot);
        fetch(min(blk + PFD, blk1 - 1), slot);             // PFD blocks ahead, in flight during the MFMAs below
        at_lds_barrier();

        // ---- S^T = K Q^T for two 32-key blocks
        f32x16_t s[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KD; ++ks) {
                const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(&Ks[kb * 32 + l32][ks * 16 + hl * 8]);
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[kb], 0, 0, 0);
            }
        }
        // ---- online softmax (this lane: query l32; keys kb*32 + (e/4)*8 + hl*4 + e%4).  The scale is positive,
        // so the running maximum is taken over the raw scores and the scale rides on the exponent's
        // multiply-add; keys that do not exist can only be in the last block of the range.
        if (__builtin_amdgcn_readfirstlane(k0 + AT_BKV > n_keys)) {      // scalar condition: a real branch, not 32 selects
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (k0 + kb * 32 + (e >> 2) * 8 + hl * 4 + (e & 3) >= n_keys) s[kb][e] = -INFINITY;
        }
        float mraw = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) mraw = fmaxf(mraw, s[kb][e]);
        const float2 mh = at_halves(mraw);
        const float mx = fmaxf(m_run, fmaxf(mh.x, mh.y) * scale_log2e);
        const float alpha = __builtin_amdgcn_exp2f(m_run - mx);   // first block: exp2(-inf) = 0
        float psum = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][e], scale_log2e, -mx));   // v_exp_f32: results below 2^-126 flush to 0
                s[kb][e] = p;
                psum += p;
            }
        l_run = l_run * alpha + psum;
        m_run = mx;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (i * 32 + (e >> 2) * 8 < DP) oacc[i][e] *= alpha;      // (rows past the head dim are not stored)

        // ---- O^T += V^T P^T : four 16-key steps; the key order inside a step follows the accumulator layout
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                uint4 pw;                                  // eight probabilities as packed bf16 pairs
                pw.x = f2bf2(s[kb][8 * jj + 0], s[kb][8 * jj + 1]); pw.y = f2bf2(s[kb][8 * jj + 2], s[kb][8 * jj + 3]);
                pw.z = f2bf2(s[kb][8 * jj + 4], s[kb][8 * jj + 5]); pw.w = f2bf2(s[kb][8 * jj + 6], s[kb][8 * jj + 7]);
                const bf16x8_t pf = *reinterpret_cast<bf16x8_t*>(&pw);
                const int kbase = kb * 32 + 16 * jj + hl * 4;
#pragma unroll
                for (int i = 0; i < DB; ++i) {
                    const uint2 lo = *reinterpret_cast<const uint2*>(&Vs[i * 32 + l32][kbase]);
                    const uint2 hi = *reinterpret_cast<const uint2*>(&Vs[i * 32 + l32][kbase + 8]);
                    uint4 v = make_uint4(lo.x, lo.y, hi.x, hi.y);
                    oacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8_t*>(&v), pf, oacc[i], 0, 0, 0);
                }
            }
      }
    }

    at_store(oacc, m_run, l_run, qok, splits, B, M, C, heads, b, h, sp, qrow, hl, d, out, part_o, part_ml);
}

// The same for long key ranges of heads of 40, 80 and 160: a turn of 64 (160: 32) keys at a time, with the products of other turns issued between the
// vector instructions of this turn's softmax: those of the values of the turn before, then the scores of the next turn, into the registers of this
// turn's as they are used up.  Operands come through LDS-direct loads, two or three turns ahead, and one barrier a turn.
// Bound by the instructions a wave issues (one in ~5 cycles: 172 vector, 14 matrix, 14 LDS and ~50 scalar ones a turn of 8 x 40; attention_kernel has
// 190, 14, 26 and ~70) and, with many queries, by power: the clock falls from 2.2 to 1.7 - 2.1 GHz under this kernel, so what the matrix units
// multiply counts too, and value rows past the head dim are read as zeros (left as they come, 4 % slower at 2 x 2752 queries, 9216 keys).
// us with the merge, attention_kernel and this one: 2 x 2752 queries, 9216 keys of 8 x 40 154 -> 142, 2 x 4096 x 4096 99 -> 88, 2 x 768 x 4096 29.6 -> 29.0; 2 x 2048 x 2304 of
// 8 x 80 44.3 -> 41.0; 2 x 576 x 576 of 8 x 160 23.0 -> 22.1.
// Products issued when the vector work of slot s of a turn starts.  Slots: the maximum, from `weights` on the probabilities (eight slots a 32-key block), from
// `rescale` on the rescaling.  The values' (DB a 16-key step) go out before the probabilities of their keys are overwritten and before the
// rescaling; the scores of a 32-key block of the next turn behind the last use of this turn's, whose registers they take.
constexpr int at_issued(int s, int slots, int weights, int NB, int DB, int KD) {
    const int values = 2 * NB * DB, rescale = weights + 8 * NB, v_end = NB == 2 ? weights + 8 : rescale;
    if (s < v_end) {
        const int even = (values * (s + 1) + v_end - 1) / v_end, need = s < weights ? 0 : DB * ((s - weights) / 4 + 1);
        return even > need ? even : need;
    }
    if (s < rescale) return values + (KD * (s + 1 - v_end) + 7) / 8;
    return values + (NB - 1) * KD + (KD * (s + 1 - rescale) + slots - rescale - 1) / (slots - rescale);
}
// Registers that a turn's operands go round in, `ahead` of them requested before they are needed: the first ones of the next turn must not meet the last of this.
constexpr int at_ring(int n, int ahead) {
    for (int r = ahead + 1;; ++r) {
        bool ok = true;
        for (int i = 0; i < ahead; ++i)
            for (int j = n - ahead + i + 1; j < n; ++j) ok = ok && j % r != i;
        if (ok) return r;
    }
}
template <int N, typename F> __device__ __forceinline__ void at_static_for(F&& f) {
    if constexpr (N > 0) { at_static_for<N - 1>(f); f(std::integral_constant<int, N - 1>{}); }
}

template <int D>
__global__ __launch_bounds__(256, 2) void attention_turns_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ K,
                                                           const bf16_t* __restrict__ Vt, int B, int M, int n_keys, int n_stride,
                                                           int C, float scale_log2e, int splits, int per, int nqt, int heads,
                                                           FastDiv d_nqt, FastDiv d_heads, FastDiv d_splits,
                                                           bf16_t* __restrict__ out, float* __restrict__ part_o, float* __restrict__ part_ml) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = AtTile<D>;
    constexpr int KD = T::KD, d = D, DB = T::DB, NB = T::NB, BK = T::BK, PITCH = T::PITCH, VPITCH = T::VPITCH, KL = T::KL, VL = T::VL, LPW = T::LPW;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // [VR][VB] values, [KR][KB] keys, zeros, what nobody reads

    const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto [qt, h, b, sp] = at_place(nqt, heads, B, splits, d_nqt, d_heads, d_splits);
    const int qrow = qt * AT_BQ + wave * AT_QW + l32;
    const bool qok = qrow < M;
    // turns of this split: `per` key blocks of 64, in turns of BK
    const int t0 = sp * per * (AT_BKV / BK), t1 = min((n_keys + BK - 1) / BK, t0 + per * (AT_BKV / BK)), turns = t1 - t0;

    bf16x8_t qf[KD];
    at_queries(qf, q, M, C, b, h, qrow, qok, hl, d);

    // ---- loads: KL of keys, VL of values, wave w takes every fourth from the w-th on.  K: LDS row r of a turn holds key
    // (r & 3) + 4 (r / 8 % 2) + 8 (r / 4 % 2) + 16 (r / 16), so that a lane's eight scores of a 16-key step are eight consecutive
    // keys, the operand of the second product as they stand; piece p of row r at r PITCH + p.  V^T: piece p (eight keys) of row r at
    // slot p ^ swizzle(r) of the row.  All of them unconditional: pieces that do not exist are read where one of the same
    // key or row exists (attention_keys.h), and behind the last turn the last one is read again.
    const unsigned char* src[LPW]; unsigned off[LPW];    // address of the next load: base, lane's offset from there
    unsigned put[LPW];                                   // its place
    const int partial = t1 * BK > n_keys ? t1 - 1 : -1;  // the turn that has fewer than BK keys
    auto load_of = [&](int t) { return min(wave + 4 * t, KL + VL - 1); };      // the last one several times over
    auto place = [&](int t, bool whole) {                // offsets in a turn of BK keys, in the partial one
        const int l = load_of(t), last = whole ? BK - 1 : n_keys - 1 - partial * BK;
        off[t] = l < KL ? T::key_offset(l * 64 + lane, last, C) : T::value_offset(l - KL, lane, last, n_stride);
    };
#pragma unroll
    for (int t = 0; t < LPW; ++t) {
        const int l = load_of(t);
        src[t] = reinterpret_cast<const unsigned char*>(l < KL ? K + ((size_t)b * n_keys + t0 * BK) * C + h * d : Vt + ((size_t)b * C + h * d + T::value_row(l - KL)) * n_stride + t0 * BK);
        put[t] = l < KL ? T::KEYS + l * 1024 : (l - KL) * 1024;
        place(t, t0 != partial);
    }
    // keys of turn `next` (behind the last one: that one again), values of the turn before (the first time: none)
    int next = t0;
    auto load = [&](bool first) {
#pragma unroll
        for (int t = 0; t < LPW; ++t)
            if (!first || load_of(t) < KL) __builtin_amdgcn_global_load_lds((const FISE_AS1 void*)(src[t] + off[t]), (FISE_AS3 void*)(lds + put[t]), 16, 0, 0);
#pragma unroll
        for (int t = 0; t < LPW; ++t) {
            const bool keys = load_of(t) < KL;
            src[t] += at_next_turn(keys, first, next) < t1 ? (keys ? (long long)C * (2 * BK) : 2ll * BK) : 0ll;
        }
        if (next + 1 == partial || (!first && next == partial)) {
            asm volatile("");                            // a branch, not selects
#pragma unroll
            for (int t = 0; t < LPW; ++t)
                if (at_next_turn(load_of(t) < KL, first, next) == partial) place(t, false);
        }
        ++next;
#pragma unroll
        for (int t = 0; t < LPW; ++t) {
            const bool keys = load_of(t) < KL;
            if (keys || !first) put[t] += keys ? T::KB : T::VB;
            if (put[t] >= (keys ? T::ZERO : T::KEYS)) put[t] -= keys ? T::KR * T::KB : T::VR * T::VB;
        }
    };

    f32x16_t oacc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;                // l: of this lane's half of the keys until the end

    if (turns > 0) {
        // zeros: what a head's last pieces are short of, and the values in front of the first turn
        if (tid < (T::LDS - T::ZERO) / 16) *reinterpret_cast<uint4*>(lds + T::ZERO + tid * 16) = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < T::VB / 16; e += 256)
            if (e + tid < T::VB / 16) *reinterpret_cast<uint4*>(lds + (T::VR - 1) * T::VB + (e + tid) * 16) = make_uint4(0, 0, 0, 0);
        load(true);
#pragma unroll
        for (int g = 0; g < T::AHEAD; ++g) load(false);
        // the query fragments have arrived before the loop: the compiler would otherwise wait for every load in flight in front of each turn's scores
#pragma unroll
        for (int ks = 0; ks < KD; ++ks) asm volatile("" ::"v"(qf[ks]));
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(T::AHEAD * LPW) : "memory");

        constexpr int NV = 2 * NB * DB, NM = NV + NB * KD, RA = 3, RING = at_ring(NM, RA);
        constexpr int WEIGHTS = 2 * NB + 1, RESCALE = WEIGHTS + 8 * NB, SLOTS = RESCALE + KD;
        // A turn's operands: piece 2 ks + hl of key row l32 (past the head dim: zeros), piece 2 u + hl of value row l32, behind a base that is
        // worked out once a turn.
        constexpr int VU = VPITCH % 2 ? 1 : 2 * NB;
        unsigned kget = T::KEYS, vget = (T::VR - 1) * T::VB, kat, vat[VU], vtail[VU];
        auto keys_at = [&]() { kat = kget + (unsigned)(l32 * PITCH + hl) * 16; };
        auto values_at = [&]() {
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                vat[u] = vget + (unsigned)(l32 * VPITCH + (VPITCH % 2 ? hl : (2 * u + hl) ^ T::swizzle(l32))) * 16;
                if (T::TAIL) vtail[u] = l32 < T::TAIL ? vat[u] : (unsigned)(T::ZERO - (DB - 1) * (32 * VPITCH * 16));
            }
        };
        auto read_k = [&](int kb, int ks) {
            const unsigned step = (unsigned)(kb * (32 * PITCH * 16) + ks * 32);
            const bool past = ks == KD - 1 && T::PAD && hl;
            return *reinterpret_cast<const bf16x8_t*>(lds + (past ? (unsigned)T::ZERO - step : kat) + step);
        };
        auto read_v = [&](int u, int i) { return *reinterpret_cast<const bf16x8_t*>(lds + (T::TAIL && i == DB - 1 ? vtail : vat)[VU == 1 ? 0 : u] + (VU == 1 ? u * 32 : 0) + i * (32 * VPITCH * 16)); };
        bf16x8_t frag[RING];
        f32x16_t s[NB];
        uint4 p[2 * NB];                                 // probabilities of the turn before: eight a 16-key step
#pragma unroll
        for (int u = 0; u < 2 * NB; ++u) p[u] = make_uint4(0, 0, 0, 0);
        keys_at();
        values_at();
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KD; ++ks) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k(kb, ks), qf[ks], s[kb], 0, 0, 0);
        }
        kget = T::KEYS + T::KB;
#pragma unroll
        for (int m = 0; m < RA; ++m) frag[m] = read_v(m / DB, m % DB);

        for (int t = t0; t < t1; ++t) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((T::AHEAD - 1) * LPW) : "memory");
            load(false);
            if (__builtin_amdgcn_readfirstlane(t == partial)) {
                const int left = n_keys - t * BK - hl * 8;
#pragma unroll
                for (int kb = 0; kb < NB; ++kb)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (kb * 32 + (e >> 3) * 16 + (e & 7) >= left) s[kb][e] = -INFINITY;
            }
            __builtin_amdgcn_sched_barrier(0);
            float mraw = -INFINITY, mx = 0.f, alpha = 0.f, psum = 0.f;
            at_static_for<SLOTS>([&](auto slot_) {
                constexpr int slot = decltype(slot_)::value, m0 = slot ? at_issued(slot - 1, SLOTS, WEIGHTS, NB, DB, KD) : 0, m1 = at_issued(slot, SLOTS, WEIGHTS, NB, DB, KD);
                at_static_for<m1 - m0>([&](auto m_) {
                    constexpr int m = m0 + decltype(m_)::value, r = (m + RA) % NM;
                    if constexpr (m < NV) {
                        oacc[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[m % RING], *reinterpret_cast<bf16x8_t*>(&p[m / DB]), oacc[m % DB], 0, 0, 0);
                    } else {
                        constexpr int kb = (m - NV) / KD, ks = (m - NV) % KD;
                        if constexpr (ks == 0)
#pragma unroll
                            for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
                        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[m % RING], qf[ks], s[kb], 0, 0, 0);
                    }
                    if constexpr (m + RA == NM) {
                        vget = vget == (T::VR - 1) * T::VB ? 0u : vget + T::VB;
                        values_at();
                    }
                    if constexpr (m + RA == NV) keys_at();
                    if constexpr (r < NV) frag[r % RING] = read_v(r / DB, r % DB);
                    else frag[r % RING] = read_k((r - NV) / KD, (r - NV) % KD);
                });
                if constexpr (slot < 2 * NB) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) mraw = fmaxf(mraw, s[slot / 2][slot % 2 * 8 + e]);
                } else if constexpr (slot < WEIGHTS) {
                    const float2 mh = at_halves(mraw);
                    mx = fmaxf(m_run, fmaxf(mh.x, mh.y) * scale_log2e);
                    alpha = __builtin_amdgcn_exp2f(m_run - mx);      // first turn: exp2(-inf) = 0
                    m_run = mx;
                } else if constexpr (slot < RESCALE) {
                    constexpr int g = slot - WEIGHTS, kb = g / 8, e = g % 8 * 2;
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][e], scale_log2e, -mx)), p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][e + 1], scale_log2e, -mx));      // v_exp_f32: results below 2^-126 flush to 0
                    psum += p0; psum += p1;
                    const unsigned w = f2bf2(p0, p1);
                    uint4& pu = p[g / 4];
                    if constexpr (g % 4 == 0) pu.x = w; else if constexpr (g % 4 == 1) pu.y = w; else if constexpr (g % 4 == 2) pu.z = w; else pu.w = w;
                } else {
                    constexpr int j = slot - RESCALE;    // rows past the head dim are not stored
#pragma unroll
                    for (int e = 0; e < 8; ++e) oacc[j / 2][j % 2 * 8 + e] *= alpha;
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            l_run = l_run * alpha + psum;
            kget = kget == T::ZERO - T::KB ? T::KEYS : kget + T::KB;
        }
        // values of the last turn; those of absent keys may be anything
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            uint4 v = *reinterpret_cast<uint4*>(&frag[m % RING]);
            if (m + RA < NV) frag[(m + RA) % RING] = read_v((m + RA) / DB, (m + RA) % DB);
            if (partial >= 0) {
                const int left = n_keys - partial * BK - m / DB * 16 - hl * 8;
                auto keep = [&](unsigned w, int t) { return left > t + 1 ? w : left > t ? w & 0xffffu : 0u; };
                v = make_uint4(keep(v.x, 0), keep(v.y, 2), keep(v.z, 4), keep(v.w, 6));
            }
            oacc[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8_t*>(&v), *reinterpret_cast<bf16x8_t*>(&p[m / DB]), oacc[m % DB], 0, 0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // loads behind the last turn still write the ring
    }

    at_store(oacc, m_run, l_run, qok, splits, B, M, C, heads, b, h, sp, qrow, hl, d, out, part_o, part_ml);
#endif
}

// Few queries: a workgroup of eight waves takes 32 queries of one (batch, head), and the waves deal the keys out among themselves, 32 at
// a time, so 256 keys are one trip to memory for all of them and no second launch merges key splits.  Nothing is shared between
// the waves before the end: each brings its keys into LDS of its own (LDS-direct loads, rows of 2 d contiguous bytes) and reads its values straight
// into matrix registers (16 rows of 64 bytes a load); the next keys are requested once the scores of these stand, their values once the
// products do.  The waves' partial sums meet in LDS, in wave order.
// 16 x 16 x 32 products; LDS row r of a wave holds key 8 (r / 4 % 4) + 4 (r / 16) + r % 4, so a lane's eight scores of a query are eight
// consecutive keys: the operand of the second product as they stand.
// Bound by the vector memory path, ~4 cycles per 128-byte line that a load instruction touches, and the start and the merge: see attention_few.
constexpr int AF_WAVES = 8;

template <int KD> struct FewTile {                      // KD: 16-wide steps over the head dim
    static constexpr int KS = (KD + 1) / 2, PS = 4 * KS, ITEMS = 2 * KD, SLICE = ITEMS < 10 ? ITEMS : 10;      // 32-wide steps, 16-byte segments of an LDS row; pieces of the output, summed at a time
    static constexpr int KBYTES = 32 * PS * 16;         // keys of a wave
    static constexpr int LDS = AF_WAVES * (KBYTES > SLICE * 1024 ? KBYTES : SLICE * 1024);
    // Segment p of row r holds segment p ^ swizzle(r) of its key: sixteen lanes that the LDS serves at once (rows 0-3, 12-15 of one segment, 4-11
    // of the next) meet in no bank.
    static __device__ __forceinline__ int swizzle(int r) {
        if (PS == 8) return (r >> 1) & 7;
        if (PS == 16) return r & 15;
        return ((r >> 2 ^ r >> 3) & 1) << 1 | (r >> 3 & 1);
    }
};

template <int KD, bool EXACT>
__global__ __launch_bounds__(64 * AF_WAVES, 2) void attention_few_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ K,
                                                                         const bf16_t* __restrict__ Vt, int B, int M, int n_keys, int n_stride,
                                                                         int C, int d_arg, float scale_log2e, int nqt, int heads,
                                                                         FastDiv d_nqt, FastDiv d_heads, bf16_t* __restrict__ out) {
#if defined(__HIP_DEVICE_COMPILE__)
    using T = FewTile<KD>;
    constexpr int KS = T::KS, PS = T::PS, NK = PS / 2;  // LDS-direct loads of 32 keys
    __shared__ __attribute__((aligned(16))) unsigned char keys[T::LDS];      // later the partial sums [waves][SLICE][64 lanes]
    __shared__ float2 ml[AF_WAVES][32];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // as above: the query tiles of a (batch, head) one behind the other, on one XCD
    int qt, h, b;
    {
        const int total = nqt * heads * B, chunk = total >> 3;
        int w = blockIdx.x;
        if (w < (chunk << 3)) w = (w & 7) * chunk + (w >> 3);
        const int t = (int)fdiv(w, d_nqt);
        b = (int)fdiv(t, d_heads);
        qt = w - t * nqt; h = t - b * heads;
    }
    const int d = EXACT ? KD * 16 : d_arg;
    const int nsb = (n_keys + AF_BKV - 1) / AF_BKV;
    // queries, keys and channels that do not exist lie outside the descriptors: zeros (attention_keys.h)
    const __amdgpu_buffer_rsrc_t rq = buf(q + (size_t)b * M * C + h * d, (unsigned)(M * C - h * d) * 2u);
    const unsigned char* const kp = reinterpret_cast<const unsigned char*>(K + (size_t)b * n_keys * C);
    const bf16_t* const vp = Vt + ((size_t)b * C + h * d) * n_stride;
    unsigned char* const my_keys = keys + wave * T::KBYTES;
    unsigned ok[NK];
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        const int slot = j * 64 + lane, r = slot / PS, seg = (slot % PS) ^ T::swizzle(r);
        const int key = 8 * ((r >> 2) & 3) + 4 * (r >> 4) + (r & 3);
        ok[j] = af_key_offset(key, seg, C, d);
    }
    // Requests for keys behind the last ones go out through descriptors of size zero, not behind branches: the compiler counts the loads
    // in flight by the path that has fewest, and each wait for values would wait for the next keys too.
    auto fetch_k = [&](int sb) {
        const __amdgpu_buffer_rsrc_t rk = buf(kp + af_key_base(C, h, d, sb), af_key_size(n_keys, C, h, d, sb));
#pragma unroll
        for (int j = 0; j < NK; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (__attribute__((address_space(3))) void*)(my_keys + j * 1024), 16, ok[j], 0, 0, 0);
    };
    u32x4_t vf[KD];
    const unsigned ov = af_value_row(l16, lq * 8, n_stride);
    auto fetch_v = [&](int sb) {
        const __amdgpu_buffer_rsrc_t rv = buf(vp, af_value_size(n_keys, n_stride, d, sb));
#pragma unroll
        for (int i = 0; i < KD; ++i)
            vf[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rv, af_value_offset(ov, i, n_stride, sb), 0, 0));
    };
    bf16x8_t qf[2][KS];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int c = ks * 32 + lq * 8;
            qf[t][ks] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rq, c < d ? (unsigned)((qt * 32 + t * 16 + l16) * C + c) * 2u : AF_OOB, 0, 0));
        }
    __builtin_amdgcn_sched_barrier(0);
    fetch_k(wave);
    fetch_v(wave);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qf[t][ks]));      // arrived before the loop, as above

    f32x4_t o[2][KD];
    float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < KD; ++i) o[t][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const unsigned rd = (unsigned)((l16 * PS + (lq ^ (T::swizzle(l16) & 3))) * 16), rx = (unsigned)(T::swizzle(l16) >> 2);      // place of segment 4 ks + lq: 64 (ks ^ rx) behind rd
#pragma unroll 1
    for (int sb = wave; sb < nsb; sb += AF_WAVES) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KD) : "memory");      // the keys have landed (the values were requested after them)
        f32x4_t s[2][2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
            for (int t = 0; t < 2; ++t) s[t][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                // rows 16 apart have the same swizzle
                const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(my_keys + rd + ((unsigned)ks ^ rx) * 64 + kt * (16 * PS * 16));
#pragma unroll
                for (int t = 0; t < 2; ++t) s[t][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[t][ks], s[t][kt], 0, 0, 0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0): the keys are in registers
        __builtin_amdgcn_sched_barrier(0);
        fetch_k(sb + AF_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        const int left = n_keys - sb * 32 - lq * 8;      // keys that exist from this lane's first one on
        const bool partial = sb * 32 + 32 > n_keys;      // uniform
        if (partial)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (kt * 4 + e >= left) s[t][kt][e] = -INFINITY;
        bf16x8_t pf[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float mraw = fmaxf(fmaxf(fmaxf(s[t][0][0], s[t][0][1]), fmaxf(s[t][0][2], s[t][0][3])), fmaxf(fmaxf(s[t][1][0], s[t][1][1]), fmaxf(s[t][1][2], s[t][1][3])));
            mraw = fmaxf(mraw, __shfl_xor(mraw, 16));
            mraw = fmaxf(mraw, __shfl_xor(mraw, 32));
            const float mx = fmaxf(m_run[t], mraw * scale_log2e), alpha = __builtin_amdgcn_exp2f(m_run[t] - mx);
            float psum = 0.f;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[t][kt][e], scale_log2e, -mx));
                    s[t][kt][e] = p;
                    psum += p;
                }
            psum += __shfl_xor(psum, 16);
            psum += __shfl_xor(psum, 32);
            l_run[t] = l_run[t] * alpha + psum;
            m_run[t] = mx;
#pragma unroll
            for (int i = 0; i < KD; ++i) o[t][i] *= alpha;
            uint4 pw = make_uint4(f2bf2(s[t][0][0], s[t][0][1]), f2bf2(s[t][0][2], s[t][0][3]), f2bf2(s[t][1][0], s[t][1][1]), f2bf2(s[t][1][2], s[t][1][3]));
            pf[t] = *reinterpret_cast<bf16x8_t*>(&pw);
        }
        if (partial) {                                   // values of absent keys may be anything
            auto keep = [&](unsigned w, int t) { return left > t + 1 ? w : left > t ? w & 0xffffu : 0u; };
#pragma unroll
            for (int i = 0; i < KD; ++i) vf[i] = u32x4_t{keep(vf[i].x, 0), keep(vf[i].y, 2), keep(vf[i].z, 4), keep(vf[i].w, 6)};
        }
#pragma unroll
        for (int i = 0; i < KD; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t) o[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, vf[i]), pf[t], o[t][i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_v(sb + AF_WAVES);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- sums of the waves that had keys: weights 2^(m_w - max m), then O in wave order
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // requests behind the last keys still write zeros into the wave's LDS
    if (lq == 0)
#pragma unroll
        for (int t = 0; t < 2; ++t) ml[wave][t * 16 + l16] = make_float2(m_run[t], l_run[t]);
    __syncthreads();
    f32x4_t* const part = reinterpret_cast<f32x4_t*>(keys);
    auto finish = [&](auto waves) {                      // of the first four waves or all
        constexpr int W = decltype(waves)::value;
        float own[2], inv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float2 v[W];
            float mx = -INFINITY, den = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) { v[w] = ml[w][t * 16 + l16]; mx = fmaxf(mx, v[w].x); }
#pragma unroll
            for (int w = 0; w < W; ++w) den += __builtin_amdgcn_exp2f(v[w].x - mx) * v[w].y;      // a wave without keys: weight 0
            own[t] = __builtin_amdgcn_exp2f(m_run[t] - mx); inv[t] = 1.0f / den;
        }
#pragma unroll
        for (int g0 = 0; g0 < T::ITEMS; g0 += T::SLICE) {       // piece g: 16 channels g / 2 of query tile g % 2
            if (g0) __syncthreads();
            if (wave < W)
#pragma unroll
                for (int g = g0; g < g0 + T::SLICE && g < T::ITEMS; ++g) part[(wave * T::SLICE + g - g0) * 64 + lane] = o[g & 1][g >> 1] * own[g & 1];
            __syncthreads();
            for (int g = g0 + wave; g < g0 + T::SLICE && g < T::ITEMS; g += AF_WAVES) {
                f32x4_t v = part[(g - g0) * 64 + lane];
#pragma unroll
                for (int w = 1; w < W; ++w) v += part[(w * T::SLICE + g - g0) * 64 + lane];
                const int m = qt * 32 + (g & 1) * 16 + l16, c = (g >> 1) * 16 + lq * 4;
                const float iv = g & 1 ? inv[1] : inv[0];
                if (m < M && c < d) *reinterpret_cast<uint2*>(out + ((size_t)b * M + m) * C + h * d + c) = make_uint2(f2bf2(v[0] * iv, v[1] * iv), f2bf2(v[2] * iv, v[3] * iv));
            }
        }
    };
    if (nsb <= 4) finish(std::integral_constant<int, 4>{}); else finish(std::integral_constant<int, AF_WAVES>{});
#endif
}

// out[b,m,c] = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^(m_s - max_s m_s), splits visited in index order.
// One thread per four channels (d is a multiple of 8: the four share a head, hence the weights).  Bound by its launch and its trips to memory: the parts
// of all splits, N at most, are requested together with their weights, one trip, and the positions come from 32-bit divisions.  us with the attention in
// front: weights and parts one behind the other; six together and the others in rounds of eight weights and four parts; this: 2 x 32 queries, 4096 keys of
// 8 x 40 (16 splits) 11.9, 12.7, 10.5; 9216 keys (29) 19.3, 19.6, 16.5; 2 x 96 x 2304 of 8 x 80 (12) 15.1, 15.7, 13.4; 2 x 192 x 9216 of 8 x 40 (16) 24.9, 25.9, 23.9.
template <int N>
__global__ __launch_bounds__(256) void attention_merge_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                              int B, int M, int C, int heads, FastDiv d_C4, FastDiv d_M, FastDiv d_d, int splits,
                                                              bf16_t* __restrict__ out) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x, row = fdiv(i, d_C4);
    if (row >= (unsigned)B * (unsigned)M) return;
    const int c = (int)(i - row * (unsigned)(C / 4)) * 4, b = (int)fdiv(row, d_M), m = (int)row - b * M;
    const int h = (int)fdiv((unsigned)c, d_d);
    const size_t ml_stride = (size_t)B * heads * M * 2, o_stride = (size_t)B * M * C;
    const float* ml0 = part_ml + (((size_t)b * heads + h) * M + m) * 2;
    const float* o0 = part_o + (size_t)row * C + c;
    float2 ml[N]; float4 o[N];
#pragma unroll
    for (int s = 0; s < N; ++s) {                        // past the last split: the last one again, not used
        const int sp = min(s, splits - 1);
        ml[s] = *reinterpret_cast<const float2*>(ml0 + sp * ml_stride);
        o[s] = *reinterpret_cast<const float4*>(o0 + sp * o_stride);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < N; ++s) mx = fmaxf(mx, ml[s].x);
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    float den = 0.f;
#pragma unroll
    for (int s = 0; s < N; ++s)
        if (s < splits) {
            const float w = __builtin_amdgcn_exp2f(ml[s].x - mx);  // an empty split has m = -inf: weight 0
            num.x += w * o[s].x; num.y += w * o[s].y; num.z += w * o[s].z; num.w += w * o[s].w;
            den += w * ml[s].y;
        }
    const float inv = 1.0f / den;
    *reinterpret_cast<uint2*>(out + (size_t)row * C + c) = make_uint2(f2bf2(num.x * inv, num.y * inv), f2bf2(num.z * inv, num.w * inv));
}

template <int D>
static int launch_turns(const void* q, const void* K, const void* Vt, int B, int M, int n_keys, int n_stride, int C, int heads, float scale, int splits,
                        void* out, float* part_o, float* part_ml, hipStream_t st) {
    constexpr int lds = AtTile<D>::LDS;
    static_assert(lds <= 80 * 1024, "two workgroups per CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attention_turns_kernel<D>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return fail(FISE_ERR_HIP, "attention: cannot raise the dynamic LDS limit");
    const int nqt = ceil_div(M, AT_BQ);
    hipLaunchKernelGGL((attention_turns_kernel<D>), dim3((unsigned)(nqt * heads * B * splits)), dim3(256), lds, st, (const bf16_t*)q, (const bf16_t*)K,
                       (const bf16_t*)Vt, B, M, n_keys, n_stride, C, scale * 1.4426950408889634f, splits, ceil_div(ceil_div(n_keys, AT_BKV), splits), nqt, heads,
                       fast_div(nqt), fast_div(heads), fast_div(splits), (bf16_t*)out, part_o, part_ml);
    return FISE_OK;
}

template <int KD, int DB, bool EXACT>
static void launch_at(const void* q, const void* K, const void* Vt, int B, int M, int n_keys, int n_stride, int C, int heads,
                      int d, float scale, int splits, void* out, float* part_o, float* part_ml, hipStream_t st) {
    if (splits == 0) {
        const int nqt = ceil_div(M, AF_BQ);
        hipLaunchKernelGGL((attention_few_kernel<KD, EXACT>), dim3((unsigned)(nqt * heads * B)), dim3(64 * AF_WAVES), 0, st, (const bf16_t*)q,
                           (const bf16_t*)K, (const bf16_t*)Vt, B, M, n_keys, n_stride, C, d, scale * 1.4426950408889634f, nqt, heads, fast_div(nqt),
                           fast_div(heads), (bf16_t*)out);
        return;
    }
    const int nqt = ceil_div(M, AT_BQ);
    dim3 grid((unsigned)(nqt * heads * B * splits));
    hipLaunchKernelGGL((attention_kernel<KD, DB, EXACT>), grid, dim3(256), 0, st, (const bf16_t*)q, (const bf16_t*)K,
                       (const bf16_t*)Vt, B, M, n_keys, n_stride, C, d, scale * 1.4426950408889634f, splits, nqt, heads,
                       fast_div(nqt), fast_div(heads), fast_div(splits), 65536 / (d / 8) + 1,
                       (bf16_t*)out, part_o, part_ml);
}

size_t attention_workspace_bytes(int B, int M, int n_keys, int C, int heads) {
    const int s = attention_splits(B, M, n_keys, C, heads);
    if (s <= 1) return 0;
    return align256((size_t)s * B * M * C * sizeof(float)) + align256((size_t)s * B * heads * M * 2 * sizeof(float));
}

int launch_attention(const void* q, const void* K, const void* Vt, int B, int M, int n_keys, int n_stride, int C, int heads,
                     float scale, void* out, void* ws, size_t ws_bytes, hipStream_t st) {
    if (M <= 0) return FISE_OK;
    const int d = C / heads;
    const int kd = ceil_div(d, 16);
    const int splits = attention_form(B, M, n_keys, n_stride, C, heads, ws && ws_bytes >= attention_workspace_bytes(B, M, n_keys, C, heads));
    float* part_o = (float*)ws;
    float* part_ml = splits > 1 ? (float*)((char*)ws + align256((size_t)splits * B * M * C * sizeof(float))) : nullptr;
    {
    ProfileScope prof(PROF_ATTENTION, 4.0 * B * (double)M * n_keys * C,
                      2.0 * ((double)B * n_keys * C * 2 + 2.0 * B * M * C), st);
#define FISE_AT(KDV, DBV) launch_at<KDV, DBV, false>(q, K, Vt, B, M, n_keys, n_stride, C, heads, d, scale, splits, out, part_o, part_ml, st)
#define FISE_AT_EXACT(KDV, DBV) launch_at<KDV, DBV, true>(q, K, Vt, B, M, n_keys, n_stride, C, heads, d, scale, splits, out, part_o, part_ml, st)
#define FISE_AT_TURNS(DV) { if (int e = launch_turns<DV>(q, K, Vt, B, M, n_keys, n_stride, C, heads, scale, splits, out, part_o, part_ml, st)) return e; }
    if (attention_turns(n_keys, n_stride, d, splits)) {
        if (d == 40) FISE_AT_TURNS(40)
        else if (d == 80) FISE_AT_TURNS(80)
        else FISE_AT_TURNS(160)
    }
    else if (kd <= 1) FISE_AT(1, 1);
    else if (kd == 2) FISE_AT(2, 1);
    else if (kd == 3) FISE_AT(3, 2);
    else if (kd == 4) FISE_AT(4, 2);
    else if (d == 80) FISE_AT_EXACT(5, 3);
    else if (kd == 5) FISE_AT(5, 3);
    else if (kd == 6) FISE_AT(6, 3);
    else if (kd <= 8) FISE_AT(8, 4);
    else if (d == 160) FISE_AT_EXACT(10, 5);
    else if (kd <= 10) FISE_AT(10, 5);
    else return fail(FISE_ERR_SHAPE, "attention: head dim %d > 160", d);
#undef FISE_AT
#undef FISE_AT_EXACT
#undef FISE_AT_TURNS
    }
    FISE_CHECK_LAUNCH("attention");
    if (splits > 1) {
        const long long n = (long long)B * M * (C / 4);
        ProfileScope prof(PROF_ATTENTION_MERGE, 0.0, (double)splits * B * M * C * 4.0 + 2.0 * B * M * C, st);
        // fewer than 2^23 threads: a split launch has at most 640 workgroups' queries
#define FISE_MERGE(N) hipLaunchKernelGGL(attention_merge_kernel<N>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part_o, part_ml, B, M, C, \
                                         heads, fast_div(C / 4), fast_div(M), fast_div(d), splits, (bf16_t*)out)
        switch (at_merge(splits)) {
            case 6: FISE_MERGE(6); break;
            case 8: FISE_MERGE(8); break;
            case 12: FISE_MERGE(12); break;
            case 16: FISE_MERGE(16); break;
            default: FISE_MERGE(AT_MAX_SPLITS);
        }
#undef FISE_MERGE
        FISE_CHECK_LAUNCH("attention merge");
    }
    return FISE_OK;
}

}  // namespace fise

using namespace fise;

extern "C" size_t fise_attention_active_workspace_bytes(int B, int M, int n_keys, int C, int heads) {
    if (B < 1 || M < 1 || n_keys < 1 || C < 1 || heads < 1) return 0;
    return attention_workspace_bytes(B, M, n_keys, C, heads);
}

extern "C" int fise_attention_active(const void* q, const void* K, const void* Vt, int dtype, int B, int M, int n_keys,
                                     int n_stride, int C, int heads, float scale, void* out, void* workspace,
                                     size_t workspace_bytes, void* stream) {
    if (!q || !K || !Vt || !out) return fail(FISE_ERR_NULL, "fise_attention_active: null pointer");
    if (dtype != FISE_BF16) return fail(FISE_ERR_DTYPE, "fise_attention_active: bf16 only (dtype %d)", dtype);
    if (B < 1 || M < 0 || n_keys < 1 || C < 1 || heads < 1 || C % heads) return fail(FISE_ERR_SHAPE, "fise_attention_active: B%d M%d keys%d C%d heads%d", B, M, n_keys, C, heads);
    const int d = C / heads;
    if (d % 8 || d > 160) return fail(FISE_ERR_SHAPE, "fise_attention_active: head dim %d (multiple of 8, <= 160)", d);
    if (n_stride < n_keys || n_stride % 8) return fail(FISE_ERR_ALIGN, "fise_attention_active: n_stride %d (>= n_keys, multiple of 8)", n_stride);
    if (!aligned16(q) || !aligned16(K) || !aligned16(Vt) || !aligned16(out) || (workspace && !aligned16(workspace)))
        return fail(FISE_ERR_ALIGN, "fise_attention_active: pointers must be 16-byte aligned");
    return launch_attention(q, K, Vt, B, M, n_keys, n_stride, C, heads, scale, out, workspace, workspace_bytes, as_stream(stream));
}
