"""The loads of attention_turns_kernel stay inside the caller's buffers and bring every existing key and value to the place its products read it from, and
its LDS reads stay inside the workgroup's: the kernel's own expressions (csrc/attention_keys.h), compiled for the host and walked turn by turn."""
import os
import subprocess


from paper_2305_17423_amd import build

HEADER = os.path.join(build.CSRC, "attention_keys.h")
# Two batch elements of two heads; the last head of the last element, whose ends are the buffers' ends.  Prints what is wrong.
PROGRAM = r"""
#include <cstdio>
#include <map>
#include "%s"
using namespace fise;
template <int D> void run(int n, int splits, int spare) {
    using T = AtTile<D>;
    const int d = D, C = 2 * d, b = 1, h = 1, stride = (n + 7) / 8 * 8 + spare;
    const long long k_end = 2ll * n * C * 2, v_end = 2ll * C * stride * 2;
    const int nblocks = (n + AT_BKV - 1) / AT_BKV, per = (nblocks + splits - 1) / splits;
    auto bad = [&](const char* what, int t, int l, int lane) { std::printf("%%s: d %%d keys %%d splits %%d turn %%d load %%d lane %%d\n", what, d, n, splits, t, l, lane); };
    for (int sp = 0; sp < splits; ++sp) {
        const int full = (n + T::BK - 1) / T::BK, end = (sp + 1) * per * (AT_BKV / T::BK), t0 = sp * per * (AT_BKV / T::BK), t1 = full < end ? full : end;
        const int partial = t1 * T::BK > n ? t1 - 1 : -1;
        for (int l = 0; l < T::KL + T::VL && t0 < t1; ++l) {
            const bool keys = l < T::KL;
            int turn = t0; bool whole = t0 != partial;
            for (int g = 0, next = t0; g < t1 - t0 + T::AHEAD + 1; ++g, ++next) {           // the groups of loads of a workgroup
                const int want = keys ? next : g ? next - 1 : t0;
                if (turn != (want < t1 ? want : t1 - 1) || whole != (turn != partial)) bad("turn", turn, l, 0);
                const int last = whole ? T::BK - 1 : n - 1 - partial * T::BK;
                for (int lane = 0; lane < 64; ++lane) {
                    const unsigned off = keys ? T::key_offset(l * 64 + lane, last, C) : T::value_offset(l - T::KL, lane, last, stride);
                    const long long base = keys ? (((long long)b * n + turn * T::BK) * C + h * d) * 2 : (((long long)b * C + h * d + T::value_row(l - T::KL)) * stride + turn * T::BK) * 2;
                    if (base + off < 0 || base + off + 16 > (keys ? k_end : v_end)) bad("outside", turn, l, lane);
                    // content: LDS piece -> (key, channel piece) / (row, chunk of keys)
                    const int slot = (keys ? l : l - T::KL) * 64 + lane;
                    if (keys) {
                        const int r = slot / T::PITCH, c = slot %% T::PITCH;
                        if (r >= T::BK || c >= d / 8) continue;
                        const int r16 = r & 15, key = (r & ~15) + (r16 < 4 ? r16 : r16 < 8 ? r16 + 4 : r16 < 12 ? r16 - 4 : r16);
                        if (turn * T::BK + key < n && base + off != (((long long)b * n + turn * T::BK + key) * C + h * d + c * 8) * 2) bad("key", turn, l, lane);
                    } else {
                        const int r = slot / T::VPITCH, c = T::VPITCH %% 2 ? slot %% T::VPITCH : (slot %% T::VPITCH) ^ T::swizzle(r);
                        if (r >= d || c >= 4 * T::NB) continue;
                        if (turn * T::BK + c * 8 < n && base + off != (((long long)b * C + h * d + r) * stride + turn * T::BK + c * 8) * 2) bad("value", turn, l, lane);
                    }
                }
                const int to = at_next_turn(keys, g == 0, next);
                if (to < t1) ++turn;
                if (to == partial) whole = false;
            }
        }
    }
    // the furthest that the products read in LDS: the head's rows of the last slot's values, all rows of the last slot's keys, the zeros behind those
    const int v_rows = T::TAIL ? d : 32 * T::DB, zeros = T::LDS - T::ZERO;
    const int v_last = (T::VR - 1) * T::VB + ((v_rows - 1) * T::VPITCH + 4 * T::NB - 1) * 16 + 16;
    const int k_last = T::KEYS + (T::KR - 1) * T::KB + ((T::BK - 1) * T::PITCH + (T::PAD ? d / 8 : 2 * T::KD) - 1) * 16 + 16;
    const int z_last = T::TAIL ? (T::VPITCH %% 2 ? 2 * (2 * T::NB - 1) * 16 : 0) + 16 : 0;          // value rows past the head: the base, the steps behind it
    if (v_last > T::KEYS || k_last > T::ZERO || z_last > zeros || (T::PAD && zeros < 16) || T::LDS > 80 * 1024) bad("LDS", 0, 0, 0);
    if (v_rows != d || (T::PAD ? 2 * T::KD * 8 != d + 8 : 2 * T::KD * 8 != d)) bad("head dim", 0, 0, 0);
    // sixteen lanes that the LDS serves together read from sixteen different groups of four banks
    for (int g = 0; g < 2; ++g) {
        unsigned seen_k = 0, seen_v = 0;
        for (int i = 0; i < 16; ++i) {
            const int even[16] = {0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27}, odd[16] = {4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31};
            const int r = g ? odd[i] : even[i];
            seen_k |= 1u << (r * T::PITCH & 15);
            seen_v |= 1u << ((r * T::VPITCH + (T::VPITCH %% 2 ? 0 : T::swizzle(r))) & 15);
        }
        if (seen_k != 0xffffu || seen_v != 0xffffu) bad("banks", 0, 0, g);
    }
}
int main() {
    const int ns[] = {1, 7, 8, 9, 31, 32, 33, 57, 63, 64, 65, 96, 97, 120, 127, 128, 129, 192, 200, 257, 320, 449};
    for (int n : ns)
        for (int splits = 1; splits <= 4; ++splits)
            for (int spare = 0; spare < 2; ++spare) {
                const int s = spare * 24;
                run<40>(n, splits, s); run<80>(n, splits, s); run<160>(n, splits, s);
            }
    std::printf("done\n");
}
"""


def test_loads_and_lds_reads(tmp_path):
    src, exe = tmp_path / "turns.cpp", tmp_path / "turns"
    src.write_text(PROGRAM % HEADER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert out == ["done"], out[:20]
