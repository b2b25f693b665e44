// Which kernel an attention launch takes and into how many parts it splits its keys: plain C++, so that a host program can ask for the form of any
// size.  Internal.
#pragma once
#include <algorithm>
#include <cmath>
#include "attention_keys.h"

namespace fise {

constexpr int AT_BQ = 128, AF_BQ = 32;        // queries of a workgroup of attention_kernel, of attention_few_kernel
constexpr int AT_MAX_SPLITS = 32;
constexpr int at_ceil(int a, int b) { return (a + b - 1) / b; }

// Key splits that the scratch of a launch is laid out for; how many it uses is attention_launch_splits' choice.  A split pays a second launch for the
// merge and, with it, ~2 us per million parked elements (rows x channels x splits); it saves key blocks, which cost a workgroup 0.9 us (head
// dim 40) to 2 us (160).  Below six blocks that never pays (four blocks of 8 x 160 channels: 2 x 32 queries 11.4 us, two splits 10.8; 2 x 192 13.8
// against 14.8; head dim 40 6.4 against 7.8).  Six and seven blocks of wide heads were worth three splits with few queries (2 x 32 queries of 8 x
// 160 channels 15.5 us unsplit, 11.4 split) before attention_few_kernel, which has those launches now: none uses that scratch, whose size callers see.
inline int attention_splits(int B, int M, int n_keys, int C, int heads) {
    const int wgs = at_ceil(M, AT_BQ) * heads * B;
    const int nblocks = at_ceil(n_keys, AT_BKV);
    if (nblocks < 6 || (nblocks < 8 && (long long)B * M * C > (C / heads - 64) * 7000LL)) return 1;
    int s = at_ceil(640, wgs);
    s = std::min(s, nblocks / 2);
    return std::max(1, std::min(s, AT_MAX_SPLITS));
}

// Parts that the merge of `splits` requests at once (loads past the last split go to that one again: not many more than there are).
constexpr int at_merge(int splits) { return splits <= 6 ? 6 : splits <= 8 ? 8 : splits <= 12 ? 12 : splits <= 16 ? 16 : AT_MAX_SPLITS; }

// What a launch costs in us, by lines fitted to 500 of attention_kernel (32 to 4096 queries, 128 to 9216 keys, heads of 40, 80 and 160, cold keys, every
// split that the scratch allows), before its turns and the present merge; d = head dim.  A workgroup spends 0.52 + 0.009 d on each of its key blocks and 0.44 more for every further
// workgroup on its CU, which holds three of heads up to 64 and two of wider ones; more workgroups than that go round again.  A split costs
// 3.5 for the merge and 2.6 per million parked elements (rows x channels x splits).
inline double attention_us(int B, int M, int n_keys, int C, int heads, int splits) {
    const int d = C / heads, resident = d <= 64 ? 3 : 2;
    const double wgs = (double)at_ceil(M, AT_BQ) * heads * B * splits;
    const double on_cu = std::min(std::ceil(wgs / 256.0), (double)resident);
    const int per = at_ceil(at_ceil(n_keys, AT_BKV), splits);
    return 2.2 + 0.0068 * d + (n_keys % AT_BKV ? 0.47 + 0.0036 * d : 0.0) +
           per * std::max(1.0, wgs / (256.0 * resident)) * (0.52 + 0.0086 * d + 0.44 * (on_cu - 1.0)) +
           (splits > 1 ? 3.5 + 2.6e-6 * splits * B * M * C : 0.0);
}

// Splits of a launch, of the `most` that its scratch holds (2.5 workgroups per CU): as many as pay for what they park.  With the kernels as they are the form
// chosen here and in attention_few is 1.3 % from the best one on average over 98 shapes (one to four batch elements, 32 to 4096 queries, 512 to 9216 keys, heads of 40, 80 and 160), 19 % at worst:
// 2 x 1376 queries, 2304 keys of 8 x 80 46.6 us in three, 39.4 in one; 4096 keys 67.5 in three, 57.0 in four; 2304 keys of 8 x 160 76.5 in three, 65.3 in two.  All
// of `most` was 11 % and 43 %.
inline int attention_launch_splits(int B, int M, int n_keys, int C, int heads, int most) {
    int best = 1;
    double us = attention_us(B, M, n_keys, C, heads, 1);
    for (int s = 2; s <= most; ++s) {
        const double t = attention_us(B, M, n_keys, C, heads, s);
        if (t < us) { us = t; best = s; }
    }
    return best;
}

// Which kernel: the one whose time is smaller, 0.6 % from the better one on average over 105 shapes, 14 % at worst.  Few queries: 2.8 + 0.019
// d us, 0.32 + 0.02 d per 256 keys and round of 256 workgroups, 0.037 d per further round.  2 x 48 queries, 256 keys of 8 x 160 channels
// 12.0 -> 10.4 us; 2 x 192 x 77 keys of 8 x 80 6.6 -> 5.4; 2 x 384 x 1024 17.0 -> 12.7; 2 x 768 x 4096 of 8 x 40 stays (31 against 36).
inline bool attention_few(int B, int M, int n_keys, int n_stride, int C, int heads, int splits) {
    const double lim = 1u << 30;                         // 32-bit offsets into a batch element
    if ((double)n_keys * C >= lim || (double)C * n_stride >= lim || (double)M * C >= lim) return false;
    const int d = C / heads, few_wgs = at_ceil(M, AF_BQ) * heads * B, rounds = at_ceil(few_wgs, 256);
    const double few = 2.8 + 0.019 * d + rounds * (at_ceil(n_keys, AF_BKV) / 8.0) * (0.32 + 0.02 * d) + (rounds - 1) * 0.037 * d;
    return few < attention_us(B, M, n_keys, C, heads, splits);
}

// Whether a launch in `splits` parts runs on attention_turns_kernel: from twelve key blocks a part on (heads of 160: eight), below which its longer set-up (1.1 us) costs more
// than its turns save.  Its time over attention_kernel's at 8, 10, 12, 16 and 20 blocks a part: heads of 40, one workgroup on a CU 1.03, 1.02, 1.00, 0.98, 0.97,
// more 1.02, 1.00, 1.00, 0.98, 0.97; of 80 1.05, 1.03, 1.00, 0.98, 0.965, more 1.00, 0.985, 0.98, 0.96, 0.95; of 160 0.97 at eight and 0.95 at ten.  Heads of
// 104 and 128 would lose (2 x 700 x 1500 of 4 x 104 31 and 33 us).  Its offsets reach over sixteen value rows in 32 bits.
inline bool attention_turns(int n_keys, int n_stride, int d, int splits) {
    return splits > 0 && (d == 40 || d == 80 || d == 160) && at_ceil(at_ceil(n_keys, AT_BKV), splits) >= (d == 160 ? 8 : 12) && n_stride < 1 << 27;
}

// Form of a launch: 0 attention_few_kernel (one launch whatever the key range), else the key splits of attention_kernel.
inline int attention_form(int B, int M, int n_keys, int n_stride, int C, int heads, bool scratch) {
    const int most = scratch ? attention_splits(B, M, n_keys, C, heads) : 1;         // what the scratch is laid out for
    const int splits = attention_launch_splits(B, M, n_keys, C, heads, most);
    return attention_few(B, M, n_keys, n_stride, C, heads, splits) ? 0 : splits;
}

// ---- cross.hip: a cross-attention sub-layer over the few keys of a prompt, `Ma` rows of a batch element of maps of HW pixels.  CROSS_LAYER: one launch;
// CROSS_QUERIES: one launch up to the last product; CROSS_STEPS: a launch each for queries, attention and product.
constexpr int CROSS_C = 320, CROSS_HEADS = 8, CROSS_KEYS = 80, CROSS_ROWS = 32;
enum { CROSS_STEPS = 0, CROSS_QUERIES = 1, CROSS_LAYER = 2 };
inline int cross_form(int C, int heads, int n_ctx, int n_stride, int B, int Ma, int HW) {
    if (heads != CROSS_HEADS || n_ctx < 1 || n_ctx > CROSS_KEYS || Ma < 1) return CROSS_STEPS;
    if (n_stride >= 1 << 20 || Ma >= 1 << 20 || HW >= 1 << 21 || (long long)B * Ma >= 1 << 24 || (long long)B * HW >= 1 << 24) return CROSS_STEPS;       // 32-bit offsets
    const long long tiles = (long long)B * at_ceil(Ma, CROSS_ROWS);
    // From forty workgroups on: with fewer, a workgroup per head and a product behind it spread the weights over more CUs.  Step of 64 x 64 with 24 workgroups
    // 1952 us as one launch and 1939 as two, with 48 2199 and 2206, with 96 2726 and 2761; attention layer of 640 rows (20) 44.8 and 43.0, of 1280 (40) 50.7 and 51.2,
    // of 4096 (128) 81.3 and 89.2.
    if (C == CROSS_C) return tiles >= 40 ? CROSS_LAYER : CROSS_QUERIES;
    // A workgroup per head and tile: one round of the CUs.  In a second one the rows are normalised too often (layer as three launches and as two, us: 992 rows
    // 22.5, 17.3, 1056 22.8, 24.4, 1536 24.9, 26.3, 2048 28.7 both; 64 batch elements of nine rows 20.7, 22.5).
    return C == 2 * CROSS_C && tiles * CROSS_HEADS <= 256 ? CROSS_QUERIES : CROSS_STEPS;
}

}  // namespace fise
