// Sum of many values with every addition rounded in index order, by one wave: plain C++ over a wave of any kind, so that a host program can run it on
// 64 lanes of its own.  Internal.
#pragma once

namespace fise {

inline constexpr double os_from_bits(long long b) { return __builtin_bit_cast(double, b); }

// s + src[0] + src[1] + ...; 0 <= values < top, no subnormals (or NaN: the sum is).  While the sum stays in one binade [2^e, 2^(e+1)) it is a
// multiple of its last place, and an addition moves it by the value rounded to a multiple of that: they add up exactly in any order.  So a block of 256
// values, four a lane, is rounded in parallel (added to 1.5 x 2^e and taken back) and scanned.  The first lane in which the sum reaches the next
// binade, or a value lies half way between two places (then the sum's last bit decides), adds its four values one by one, and the scan goes on
// behind it, moved by what those values made of it.  Sums of the scan past the binade are rounded to its coarser places: nothing but that they lie
// there is taken from them, so where any lane's does, the lanes behind one that was added by itself are scanned afresh.  Blocks with many such values, and values
// of 2^(e-1) and more, are added one by one.
// Wave: Lanes, a double for each lane, with arithmetic and comparisons; ballot of a comparison; at(x, lane); from(x, lane): x in this lane and those behind it, else zero; scan: sums
// over the lanes up to each, of which those that a binade holds are exact; before(x): the lane in front's; load(src, i, total): src[i + 4 lane + 0 .. 3], zeros behind `total`;
// uniform: a value that all lanes agree on.
template <class Wave>
#if defined(__HIPCC__)
__device__
#endif
inline double ordered_sum(double s, const double* src, int total, double top) {
    using Lanes = typename Wave::Lanes;
    constexpr int Q = 4, BLOCK = 64 * Q, HEAD = 8, TIES = 8;   // HEAD: lanes of the first values, which change the binade all the time
    Lanes v[Q], next[Q];
    auto take = [&](int at) {
#pragma unroll
        for (int q = 0; q < Q; ++q) s += Wave::at(v[q], at);
    };
    if (total > 0) Wave::load(next, src, 0, total);
    for (int i0 = 0; i0 < total; i0 += BLOCK) {
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = next[q];
        Wave::load(next, src, i0 + BLOCK, total);
        int done = 0, ties = 0;                                // lanes whose values are in the sum
        const int left = (total - i0 + Q - 1) / Q, lanes = left < 64 ? left : 64;
        if (i0 == 0)
            for (; done < lanes && done < HEAD; ++done) take(done);
        while (done < lanes) {
            const int e = Wave::uniform((int)(__builtin_bit_cast(long long, s) >> 52)) & 0x7ff;        // of a NaN whatever its sign
            if (e == 0x7ff) return s;
            const double one = os_from_bits((long long)e << 52);       // 2^e; zero: the sum is zero
            if (ties > TIES || Wave::uniform((int)(top > 0.5 * one))) {
                if (e == 0) {                                  // passes over zeros
                    const unsigned long long some = Wave::ballot(!((v[0] == 0.0) & (v[1] == 0.0) & (v[2] == 0.0) & (v[3] == 0.0))) & (~0ull << done);
                    if (!some) break;
                    done = __builtin_ctzll(some);
                }
                const int until = lanes < done + HEAD ? lanes : done + HEAD;
                for (; done < until; ++done) take(done);
                continue;
            }
            const double grid = 1.5 * one, half = one * 0x1p-53, end = 2.0 * one;
            Lanes run = Wave::zero();
            unsigned long long tie = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const Lanes r = (v[q] + grid) - grid;
                tie |= Wave::ballot(!(Wave::abs(v[q] - r) < half));     // NaN too
                run = run + r;
            }
            run = Wave::from(run, done);
            Lanes base = Wave::before(Wave::scan(run)) + s;    // the sum in front of each lane
            for (;;) {
                const unsigned long long past = Wave::ballot(!(base + run < end)), stop = (tie | past) & (~0ull << done);
                if (!stop) { s = Wave::at(base + run, 63); done = 64; break; }
                const int at = __builtin_ctzll(stop);
                const double here = Wave::at(base + run, at);
                s = Wave::at(base, at);
                take(at);
                done = at + 1;
                if (done >= lanes || Wave::uniform((int)!(s < end)) || ++ties > TIES || past & (~0ull << done)) break;      // another binade, here or further on
                base = base + (s - here);
            }
        }
    }
    return s;
}

}  // namespace fise
