// Sum of many values with every addition rounded in index order, by one wave: plain C++ over a wave of any kind, so that a host program can run it on
// 64 lanes of its own.  Internal.
#pragma once

#if defined(__HIPCC__)
#define FISE_OS_FN __device__ __forceinline__
#else
#define FISE_OS_FN inline
#endif

namespace fise {

// s + src[0] + src[1] + ...; 0 <= values <= 1, no subnormals (or NaN: the sum is).  While the sum stays in one binade [2^e, 2^(e+1)) it is a
// multiple of its last place, and an addition moves it by the value rounded to a multiple of that: they add up exactly in any order.  So a block of 256
// values, four a lane, is rounded in parallel (added to 1.5 x 2^e and taken back) and scanned.  The scan stops at the first lane in which the sum
// reaches the next binade, a value lies half way between two places (then the sum's last bit decides) or the four are over 2^(e-1) (values that large are
// not rounded as the sum would be); that lane's four values are added one by one, and the scan goes on behind it, moved by what they made of it.  Sums of the scan past the binade are
// rounded to its coarser places: nothing but that they lie there is taken from them, so where any lane's does, the lanes behind one that was added by
// itself are scanned afresh.  A block with more such lanes than a few is added one by one, and so are once, three times, seven times ... as many blocks behind
// it, until a block scans.  The values themselves decide, not how large a bin's may be: one that is mostly zeros, or whose sum stays far below its values'
// bound, scans like any other.  With threshold and mask, us, one addition after the other and this: 4096 values of an edit 21.6, 18.6; of which nine in ten are zero
// 30.5, 17.2; 9216 57.4, 27.8 (68 and 186 with every sum below 2^-7 added one by one in registers); all equal 61.9, 39.8; ties throughout, 1024 values 16.7, 18.1, 4096 32.2, 30.5.
// Wave: Lanes, a double for each lane, with arithmetic and comparisons; ballot of a comparison; at(x, lane); from(x, lane): x in this lane and those behind it, else zero; scan: sums
// over the lanes up to each, of which those that a binade holds are exact; before(x): the lane in front's; load(src, i, total): src[i + 4 lane + 0 .. 3], zeros behind `total`;
// uniform: a value that all lanes agree on.  Src: the values, 16 zeros behind them and 8 more that can be read.
template <class Wave, class Src>
FISE_OS_FN double ordered_sum(double s, Src src, int total) {
    using Lanes = typename Wave::Lanes;
    constexpr int Q = 4, BLOCK = 64 * Q, HEAD = 8, STOPS = 8, AHEAD = 8;      // HEAD: lanes of the first values, which change the binade all the time
    Lanes v[Q], next[Q];
    auto take = [&](int at) {
#pragma unroll
        for (int q = 0; q < Q; ++q) s += Wave::at(v[q], at);
    };
    auto walk = [&](int i, int to) {                           // one after the other, the next eight on their way; `to`: the end or a multiple of sixteen from i
        double x[AHEAD], y[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) x[q] = src[i + q];
        for (; i < to; i += 2 * AHEAD) {
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) y[q] = src[i + AHEAD + q];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) s += x[q];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) x[q] = src[i + 2 * AHEAD + q];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) s += y[q];
        }
    };
    int one_by_one = 0, again = 0;                             // blocks still to be added one by one, as many as the last time
    if (total > 0) Wave::load(next, src, 0, total);
    for (int i0 = 0; i0 < total; i0 += BLOCK) {
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = next[q];
        Wave::load(next, src, i0 + BLOCK, total);
        const int left = total - i0, lanes = left < BLOCK ? (left + Q - 1) / Q : 64, to = left < BLOCK ? total : i0 + BLOCK;
        int done = 0, stops = 0;                               // lanes whose values are in the sum
        if (i0 == 0) {
            walk(0, to < HEAD * Q ? to : HEAD * Q);
            done = HEAD;
        } else if (one_by_one) {
            walk(i0, to);
            --one_by_one;
            continue;
        }
        const Lanes four = (v[0] + v[1]) + (v[2] + v[3]);
        const unsigned long long some = Wave::ballot(!(four == 0.0));      // lanes that change the sum
        while (done < lanes && some & (~0ull << done)) {
            const int e = Wave::uniform((int)(__builtin_bit_cast(long long, s) >> 52)) & 0x7ff;        // of a NaN whatever its sign
            if (e == 0x7ff) return s;
            if (e == 0 || stops > STOPS) {                     // nothing in the sum yet, or a block that stops too often
                done = __builtin_ctzll(some & (~0ull << done));
                for (; done < lanes && done % 4; ++done) take(done);
                const int until = stops > STOPS || done + HEAD > lanes ? lanes : done + HEAD;
                if (done < until) walk(i0 + done * Q, until < lanes ? i0 + until * Q : to);
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
            alone |= Wave::ballot(!(four <= 0.5 * one));
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
        if (stops > STOPS) one_by_one = again = 2 * again + 1; else again = 0;
    }
    return s;
}

}  // namespace fise
