"""The key addresses of the attention kernel stay inside the caller's buffers: the kernel's own expressions
(csrc/attention_keys.h), compiled for the host, over every number of keys up to a few blocks."""
import os
import subprocess

import numpy as np
import pytest

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
