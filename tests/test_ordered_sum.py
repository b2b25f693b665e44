"""The sums of the Otsu bins, rounded ahead and scanned, are the sums in index order bit for bit: the kernel's own loop (csrc/ordered_sum.h), run on 64 lanes of
the host that add up as the wavefront's do, against one addition after the other."""
import os
import subprocess

import pytest

from paper_2305_17423_amd import build

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#include "%s"
typedef unsigned long long u64;
struct Lanes { double x[64]; };
struct Flags { u64 m; };
template <class F> Lanes each(F f) { Lanes r; for (int i = 0; i < 64; ++i) r.x[i] = f(i); return r; }
template <class F> Flags where(F f) { Flags r{0}; for (int i = 0; i < 64; ++i) r.m |= (u64)f(i) << i; return r; }
Lanes operator+(const Lanes& a, const Lanes& b) { return each([&](int i) { return a.x[i] + b.x[i]; }); }
Lanes operator-(const Lanes& a, const Lanes& b) { return each([&](int i) { return a.x[i] - b.x[i]; }); }
Lanes operator+(const Lanes& a, double b) { return each([&](int i) { return a.x[i] + b; }); }
Lanes operator-(const Lanes& a, double b) { return each([&](int i) { return a.x[i] - b; }); }
Flags operator<=(const Lanes& a, double b) { return where([&](int i) { return a.x[i] <= b; }); }
Flags operator<(const Lanes& a, double b) { return where([&](int i) { return a.x[i] < b; }); }
Flags operator==(const Lanes& a, double b) { return where([&](int i) { return a.x[i] == b; }); }
Flags operator!(Flags a) { return {~a.m}; }
Flags operator&(Flags a, Flags b) { return {a.m & b.m}; }
Flags operator|(Flags a, Flags b) { return {a.m | b.m}; }
long long walked;                                        // values read one by one
struct Values { const double* v; int n; double operator[](int i) const { if (i < 0 || i >= n) std::abort(); ++walked; return v[i]; } };
struct Wave {
    using Lanes = ::Lanes;
    static Lanes zero() { return each([](int) { return 0.0; }); }
    static Lanes abs(const Lanes& a) { return each([&](int i) { return std::fabs(a.x[i]); }); }
    static u64 ballot(Flags a) { return a.m; }
    static int uniform(int x) { return x; }
    static double at(const Lanes& a, int lane) { ++walked; return a.x[lane]; }
    static Lanes from(const Lanes& a, int first) { return each([&](int i) { return i < first ? 0.0 : a.x[i]; }); }
    static Lanes before(const Lanes& a) { return each([&](int i) { return i ? a.x[i - 1] : 0.0; }); }
    static Lanes scan(Lanes a) {                         // rows of 16, then their last lanes, as the wavefront's moves do it
        for (int o = 1; o < 16; o *= 2) a = a + each([&](int i) { return i %% 16 >= o ? a.x[i - o] : 0.0; });
        a = a + each([&](int i) { return i / 16 %% 2 ? a.x[i / 16 * 16 - 1] : 0.0; });
        return a + each([&](int i) { return i >= 32 ? a.x[31] : 0.0; });
    }
    static void load(Lanes (&x)[4], const Values& src, int i0, int total) {
        for (int q = 0; q < 4; ++q) x[q] = each([&](int i) { const int at = i0 + 4 * i + q; return at < total ? src.v[at] : 0.0; });
    }
};
int main(int, char** argv) {
    const std::string_view shape = argv[1];
    const bool one_by_one_counts = argv[3][0] == '1';                  // long sums in chunks of the kernel's size
    int bad = 0, runs = std::atoi(argv[2]);
    long long all = 0;
    for (int seed = 0; seed < runs; ++seed) {
        std::mt19937_64 g(seed);
        auto unit = [&] { return (g() >> 11) * 0x1p-53; };
        const int bin = shape == "edge" || one_by_one_counts ? 0 : shape == "nan" ? (int)(g() %% 4) * 64 : (int)(g() %% 257);
        const double low = bin / 256.0, top = bin < 256 ? (bin + 1) / 256.0 : 1.0;
        std::vector<double> v;
        if (shape == "edge") {                           // up to a few places below 2, then ties and whole places across it
            v.assign(1023, 0x1p-9);
            const int k = 1 + g() %% 64;                 // 2 - k 2^-52
            const long long rest = (1ll << 43) - k;      // of 2^-9, in places of 2^-52
            for (int b = 42; b >= 0; --b) if (rest >> b & 1) v.push_back(std::ldexp(1.0, b - 52));
            v.resize((v.size() + 255) / 256 * 256);
            for (int i = 0; i < 256; ++i) v.push_back((g() %% 8 ? 0 : 1 + g() %% 6) * (g() %% 3 ? 0x1p-53 : 0x1p-52));
        } else {
            const int n = one_by_one_counts ? 4096 + (int)(g() %% 5000) : 1 + g() %% 1500;
            const double c = low + unit() / 256;
            for (int i = 0; i < n; ++i) {
                double x = low + unit() / 256;
                if (bin == 256) x = 1.0;
                if (shape == "sparse" && g() %% 10) x = 0;
                if (shape == "tiny") x = std::ldexp(unit(), -30 - (int)(g() %% 30));
                if (shape == "mixed") x = std::ldexp(x, -(int)(g() %% 60));
                if (shape == "ties") x = (double)(long long)(c * 0x1p44 + (g() %% 4)) * 0x1p-44;      // ten last bits are zero: a row of 2^9 is a tie
                if (shape == "equal") x = c;
                v.push_back(x);
            }
            if (shape == "nan") v[g() %% v.size()] = g() %% 2 ? NAN : -NAN;
        }
        // in chunks, as the kernel hands them over
        double want = 0, got = 0;
        all += v.size();
        const int chunk = g() %% 2 || one_by_one_counts ? 4096 : 700;
        for (size_t i = 0; i < v.size(); i += chunk) {
            const int n = (int)std::min<size_t>(chunk, v.size() - i);
            for (int j = 0; j < n; ++j) want += v[i + j];
            std::vector<double> part(v.begin() + i, v.begin() + i + n);
            part.resize(n + 24);
            got = fise::ordered_sum<Wave>(got, Values{part.data(), n + 24}, n, top);
        }
        if (std::memcmp(&want, &got, 8) && !(want != want && got != got) && ++bad < 4) std::printf("seed %%d: %%a, in order %%a\n", seed, got, want);
    }
    std::printf("%%d of %%d differ, %%.0f %%%% one by one\n", bad, runs, 100.0 * walked / all);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("ordered_sum")
    (d / "sum.cpp").write_text(PROGRAM % os.path.join(build.CSRC, "ordered_sum.h"))
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wno-unknown-pragmas", "-o", str(d / "sum"), str(d / "sum.cpp")], check=True)
    return str(d / "sum")


def run(program, shape, runs, long=0):
    out = subprocess.run([program, shape, str(runs), str(long)], check=True, capture_output=True, text=True).stdout
    assert out.startswith(f"0 of {runs} differ"), out
    return int(out.split(", ")[1].split()[0])


@pytest.mark.parametrize("shape,runs", [("edge", 20000), ("uniform", 1500), ("sparse", 1500), ("tiny", 1500), ("mixed", 1500), ("ties", 1500), ("equal", 1500), ("nan", 500)])
def test_sums_in_index_order(program, shape, runs):
    run(program, shape, runs)


@pytest.mark.parametrize("shape", ["uniform", "sparse", "tiny", "mixed", "equal"])
def test_long_sums_are_scanned(program, shape):
    """4096 and more values of the lowest bin, zeros, tiny and equal ones among them: few are added one by one (32 at the head, four a stop of the scan)."""
    assert run(program, shape, 200, 1) <= 15
