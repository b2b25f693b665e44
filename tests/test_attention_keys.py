"""The key addresses of the attention kernels stay inside the caller's buffers: the kernels' own expressions
(csrc/attention_keys.h), compiled for the host, over every number of keys up to a few blocks (attention of few queries: around one,
two and eight blocks, every head dim with a padding of its own)."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2305_17423_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2305_17423_amd", "csrc", "attention_keys.h")
N_KEYS = 200
# one line per (number of keys, block, key of the slot): both shifts; K slots that hold nothing carry key -1, V^T slots the
# chunk of their keys in the first row
PROGRAM = r"""
#include <cstdio>
#include "%s"
using namespace fise;
int main() {
    for (int n = 1; n <= %d; ++n)
        for (int k0 = 0; k0 < n; k0 += AT_BKV)
            for (int key = -1; key < AT_BKV; ++key) {
                const bool whole = k0 + AT_BKV <= n;
                const int last = n - 1 - k0;
                std::printf("%%d %%d %%d %%d %%d\n", n, k0, key, whole ? k0 : at_key_shift(k0, last, key), whole ? k0 : at_value_shift(k0, last, key));
            }
}
"""


@pytest.fixture(scope="module")
def shifts(tmp_path_factory):
    d = tmp_path_factory.mktemp("attention_keys")
    src, exe = d / "keys.cpp", d / "keys"
    src.write_text(PROGRAM % (HEADER, N_KEYS))
    subprocess.run(["g++", "-std=c++17", "-o", str(exe), str(src)], check=True)
    return np.array([l.split() for l in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()], np.int64)


def test_key_rows_stay_inside(shifts):
    n, k0, key, ks, _ = shifts.T
    row = np.maximum(key, 0) + ks                       # a slot that holds nothing points at row 0 of block 0
    assert (row >= 0).all() and (row < n).all()
    exists = (key >= 0) & (k0 + key < n)
    assert np.array_equal(row[exists], (k0 + key)[exists])


def test_value_chunks_stay_inside_the_shortest_row(shifts):
    s = shifts[(shifts[:, 2] >= 0) & (shifts[:, 2] % 8 == 0)]
    n, k0, key, _, vs = s.T
    first = key + vs
    stride = (n + 7) // 8 * 8                           # the smallest row an entry point accepts
    over = first + 8 - stride
    assert (first >= 0).all() and (over <= 0).all(), f"up to {over.max()} elements past a row, first at {n[over > 0][:1]} keys"
    exists = (key >= 0) & (k0 + key < n)
    assert np.array_equal(first[exists], (k0 + key)[exists]) and (first % 8 == 0).all()


def test_value_chunks_of_the_last_row_end_at_the_buffer(shifts):
    """Whole addresses, B 2, 320 channels, 8 heads: no chunk of any row leaves V^T [B, C, stride]."""
    B, C = 2, 320
    s = shifts[(shifts[:, 2] >= 0) & (shifts[:, 2] % 8 == 0)]
    n, _, key, _, vs = s.T
    stride = (n + 7) // 8 * 8
    end = (B * C - 1) * stride + key + vs + 8
    assert (end <= B * C * stride).all(), int((end - B * C * stride).max())


# Attention of few queries.  One line per 16-byte read that a lane may issue: K or V, number of keys, row stride of V^T, head dim, block (one past
# the last among them), channel segment or row, key (K: of the block; V: first of eight) and base, size of the descriptor, lane offset in bytes
# from there; two heads, the last one, whose end is the end of the batch element.
FEW = r"""
#include <cstdio>
#include "%s"
using namespace fise;
int main() {
    const int ds[] = {8, 24, 40, 56, 80, 104, 112, 136, 160}, kds[] = {1, 2, 3, 4, 5, 8, 8, 10, 10};
    const int ns[] = {1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 77, 96, 255, 256, 257};
    for (int di = 0; di < 9; ++di)
        for (int n : ns) {
            const int d = ds[di], C = 2 * d, h = 1, blocks = (n + AF_BKV - 1) / AF_BKV;
            for (int sb = 0; sb <= blocks; ++sb) {
                for (int key = 0; key < AF_BKV; ++key)
                    for (int seg = 0; seg < (kds[di] + 1) / 2 * 4; ++seg)
                        std::printf("0 %%d 0 %%d %%d %%d %%d %%u %%u %%u\n", n, d, sb, seg, key, af_key_base(C, h, d, sb), af_key_size(n, C, h, d, sb), af_key_offset(key, seg, C, d));
                for (int stride = (n + 7) / 8 * 8, wide = 0; wide < 2; ++wide, stride += 24)
                    for (int i = 0; i < kds[di]; ++i)
                        for (int r = 0; r < 16; ++r)
                            for (int q = 0; q < 4; ++q)
                                std::printf("1 %%d %%d %%d %%d %%d %%d %%u %%u %%u\n", n, stride, d, sb, i * 16 + r, q * 8, (unsigned)(h * d * stride * 2), af_value_size(n, stride, d, sb),
                                            af_value_offset(af_value_row(r, q * 8, stride), i, stride, sb));
            }
        }
}
"""


@pytest.fixture(scope="module")
def few_reads(tmp_path_factory):
    d = tmp_path_factory.mktemp("attention_few")
    src, exe = d / "few.cpp", d / "few"
    src.write_text(FEW % HEADER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), str(src)], check=True)
    return np.fromstring(subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout, np.int64, sep=" ").reshape(-1, 10)


def test_few_queries_key_reads_stay_inside(few_reads):
    """A lane offset below the descriptor's size is a read inside K [n, C] of the batch element, of exactly the keys and channels that exist."""
    s = few_reads[few_reads[:, 0] == 0]
    _, n, _, d, sb, seg, key, base, size, off = s.T
    C, live = 2 * d, off < size
    assert (base + off + 16 <= 2 * n * C)[live].all()
    assert np.array_equal(live, (sb * 32 + key < n) & (seg * 8 < d))
    assert np.array_equal((base + off)[live], (2 * ((sb * 32 + key) * C + d + seg * 8))[live])


def test_few_queries_value_reads_stay_inside(few_reads):
    """The same of V^T [C, stride]: rows of the head only, no further than its last; chunks that hold an existing key come from their place."""
    s = few_reads[few_reads[:, 0] == 1]
    _, n, stride, d, sb, row, first, base, size, off = s.T
    live, block = off < size, sb * 32 < n
    assert (base + off + 16 <= 2 * 2 * d * stride)[live].all()
    assert not live[(row >= d) | ~block].any()
    exists = (row < d) & (sb * 32 + first < n)
    assert live[exists].all() and np.array_equal((base + off)[exists], (2 * ((d + row) * stride + sb * 32 + first))[exists])


def test_few_queries_reads_have_no_scalar_offset(tmp_path):
    """What the two tests above hold is all there is: every buffer load of the kernel compares its lane offset alone with the descriptor's size."""
    out = tmp_path / "attention.s"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-x", "hip", "-S", os.path.join(build.CSRC, "attention.hip"), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernel, loads = "", {}
    for line in out.read_text().splitlines():
        if m := re.match(r"(_ZN4fise\w+):", line):
            kernel = m.group(1)
        elif "attention_few_kernel" in kernel and (m := re.match(r"\s+buffer_load_\w+ (.*)", line)):
            loads.setdefault(kernel, []).append(m.group(1).split(",")[-1].split()[0])      # "s20 offen lds": the scalar offset comes first
    assert len(loads) >= 10, sorted(loads)
    for name, offsets in loads.items():
        assert set(offsets) == {"0"}, (name, sorted(set(offsets)))
