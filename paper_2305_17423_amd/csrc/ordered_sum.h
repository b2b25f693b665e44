// Sum of many values with every addition rounded in index order, by one wave: plain C++ over a wave of any kind, so that a host program can run it on
// 64 lanes of its own.  Internal.
#pragma once

#if defined(__HIPCC__)
#define FISE_OS_FN __device__ __forceinline__
#else
#define FISE_OS_FN inline
#endif

namespace fise {

// s + src[0] + src[1] + ...; 0 <= values <= top, no subnormals (or NaN: the sum is).  While the sum stays in one binade [2^e, 2^(e+1)) it is a
// multiple of its last place, and an addition moves it by the value rounded to a multiple of that: they add up exactly in any order.  So a block of 256
// values, four a lane, is rounded in parallel (added to 1.5 x 2^e and taken back) and scanned.  The scan stops at the first lane in which the sum
// reaches the next binade, a value lies half way between two places (then the sum's last bit decides) or the four are over 2^(e-1) (values that large are
// not rounded as the sum would be); that lane's four values are added one by one, and the scan goes on behind it, moved by what they made of it.  Sums of the scan past the binade are
// rounded to its coarser places: nothing but that they lie there is taken from them, so where any lane's does, the lanes behind one that was added by
// itself are scanned afresh.  Added one by one are the first values (the sum changes its binade all the time), a block with more such lanes than a few, and what is too little for a
// scan.  A scan takes ~900 cycles, as long as 56 values one by one, a lane that stops it as long as twenty.  With threshold and mask, us, every sum one by one and this: the differences
// of five steps, 64 x 64 25.9, 21.3, 96 x 96 48.1, 34.1; nine in ten of 4096 values zero 30.4, 20.4; one bin of 9216 values 61.9, 39.6; every bin of 36 20.4, 18.3.
// (A bound of the values in the place of their own size, and register reads for what is added one by one, took 45 us for those zeros and 221 for 9216 tiny values.)  Few values of few
// bits lose up to 1.1 us to ties: one step of 32 x 48 15.7, 16.8.
// Wave: Lanes, a double for each lane, with arithmetic and comparisons; ballot of a comparison; at(x, lane); from(x, lane): x in this lane and those behind it, else zero; scan: sums
// over the lanes up to each, of which those that a binade holds are exact; before(x): the lane in front's; load(src, i, total): src[i + 4 lane + 0 .. 3], zeros behind `total`;
// uniform: a value that all lanes agree on.  Src: the values, 16 zeros behind them and 8 more that can be read.
template <class Wave, class Src>
FISE_OS_FN double ordered_sum(double s, Src src, int total, double top) {
    using Lanes = typename Wave::Lanes;
    constexpr int Q = 4, BLOCK = 64 * Q, HEAD = 32, STOPS = 8, FEW = 48, AHEAD = 8;      // HEAD: lanes of the first values, which change the binade all the time
    Lanes v[Q], next[Q];
    auto take = [&](int at) {
#pragma unroll
        for (int q = 0; q < Q; ++q) s += Wave::at(v[q], at);
    };
    auto walk = [&](int from, int to) {                        // one after the other, the next eight on their way
        int i = from & ~(AHEAD - 1);
        double x[AHEAD], y[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) { x[q] = src[i + q]; if (i + q < from) x[q] = 0.0; }       // + 0 changes no sum of values >= 0
        for (; i < to; i += 2 * AHEAD) {                       // `to`: the end or a multiple of sixteen
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) y[q] = src[i + AHEAD + q];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) s += x[q];
            if (i + AHEAD >= to) break;
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) x[q] = src[i + 2 * AHEAD + q];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) s += y[q];
        }
    };
    if (total > 0) Wave::load(next, src, 0, total);
    for (int i0 = 0; i0 < total; i0 += BLOCK) {
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = next[q];
        Wave::load(next, src, i0 + BLOCK, total);
        const int left = total - i0, lanes = left < BLOCK ? (left + Q - 1) / Q : 64, to = left < BLOCK ? total : i0 + BLOCK;
        int done = 0, stops = 0;                               // lanes whose values are in the sum
        while (done < lanes) {
            const int e = Wave::uniform((int)(__builtin_bit_cast(long long, s) >> 52)) & 0x7ff;        // of a NaN whatever its sign
            if (e == 0x7ff) return s;
            if (e == 0 || stops > STOPS || total <= FEW) {     // nothing in the sum yet, a block that stops too often, or not worth a scan
                if (i0 + done && e == 0) {                     // to the first lane with something
                    const unsigned long long some = Wave::ballot(!((v[0] + v[1]) + (v[2] + v[3]) == 0.0)) & (~0ull << done);
                    if (!some) break;
                    done = __builtin_ctzll(some);
                }
                const int until = stops > STOPS || total <= FEW ? 64 : (done + HEAD + 3) & ~3;
                walk(i0 + done * Q, until < lanes ? i0 + until * Q : to);
                done = until;
                continue;
            }
            const double one = __builtin_bit_cast(double, (long long)e << 52), grid = 1.5 * one, half = one * 0x1p-53, end = 2.0 * one;
            Lanes run = Wave::zero();
            unsigned long long alone = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const Lanes r = (v[q] + grid) - grid;
                alone |= Wave::ballot(!(Wave::abs(v[q] - r) < half));      // NaN too
                run = run + r;
            }
            if (__builtin_popcountll(alone & (~0ull << done)) > STOPS) { stops = STOPS + 1; continue; }
            if (Wave::uniform((int)(top > 0.5 * one))) alone |= Wave::ballot(!((v[0] + v[1]) + (v[2] + v[3]) <= 0.5 * one));
            run = Wave::from(run, done);
            Lanes base = Wave::before(Wave::scan(run)) + s;    // the sum in front of each lane
            for (;;) {
                const unsigned long long past = Wave::ballot(!(base + run < end)), stop = (alone | past) & (~0ull << done);
                if (!stop) { s = Wave::at(base + run, 63); done = 64; break; }
                const int at = __builtin_ctzll(stop);
                const double here = Wave::at(base + run, at);
                s = Wave::at(base, at);
                take(at);
                done = at + 1;
                if (done >= lanes || Wave::uniform((int)!(s < end)) || ++stops > STOPS || past & (~0ull << done)) break;      // another binade, here or further on
                base = base + (s - here);
            }
        }
    }
    return s;
}

}  // namespace fise
