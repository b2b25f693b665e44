"""Where the key range of the attention is split over workgroups: the scratch size tells, on the host.  Which kernel and how many splits the cases of the
GPU tests run: the launcher's own rule (csrc/attention_choice.h), compiled for the host."""
import subprocess

import pytest

import test_gpu_attention as attention
import test_gpu_cross as cross
from paper_2305_17423_amd import binding as fb, build


@pytest.mark.parametrize("B,M,n_keys,C,splits", [
    (2, 32, 320, 1280, 1),           # five blocks: one chain, whatever the head
    (1, 1, 320, 1280, 1),
    (2, 32, 321, 1280, 3),           # six and seven blocks of wide heads with few queries
    (2, 32, 448, 1280, 3),
    (2, 262, 384, 1280, 3),          # both sides of the line at head dim 160 (672000 elements), 128 and 80
    (2, 263, 384, 1280, 1),
    (2, 218, 448, 1024, 3),
    (2, 219, 448, 1024, 1),
    (2, 87, 448, 640, 3),
    (2, 88, 448, 640, 1),
    (1, 1, 448, 512, 1),             # heads of 64 and less gain nothing there
    (1, 1, 448, 320, 1),
    (2, 32, 512, 320, 4),            # eight blocks and more, any head
    (2, 4096, 512, 320, 2),
])
def test_key_splits(B, M, n_keys, C, splits):
    def up(n):
        return (n + 255) // 256 * 256
    need = up(splits * B * M * C * 4) + up(splits * B * 8 * M * 8) if splits > 1 else 0
    assert fb.fise_attention_active_workspace_bytes(B, M, n_keys, C, 8) == need


PROGRAM = r"""
#include <cstdio>
#include "%s/attention_choice.h"
int main() {
    int B, M, n, C, heads;
    while (std::scanf("%%d %%d %%d %%d %%d", &B, &M, &n, &C, &heads) == 5)
        std::printf("%%d %%d\n", fise::attention_form(B, M, n, (n + 7) / 8 * 8, C, heads, false), fise::attention_form(B, M, n, (n + 7) / 8 * 8, C, heads, true));
}
"""


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    """[(B, queries, keys, channels, heads)] -> [(without scratch, with it)]: 0 the kernel for few queries, else the splits of the one for many"""
    d = tmp_path_factory.mktemp("attention_forms")
    (d / "forms.cpp").write_text(PROGRAM % build.CSRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(d / "forms"), str(d / "forms.cpp")], check=True)

    def run(shapes):
        r = subprocess.run([str(d / "forms")], input="\n".join(" ".join(map(str, s)) for s in shapes), check=True, capture_output=True, text=True)
        return [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    return run


def test_forms_of_the_gpu_cases(forms):
    assert forms([c[:5] for c in attention.ACTIVE]) == [c[5:] for c in attention.ACTIVE]
    few = {c[3] // c[4] for c in attention.ACTIVE if c[6] == 0}
    assert {-(-d // 16) for d in few} >= {1, 2, 3, 4, 5, 6, 7, 8, 9, 10}, sorted(few)       # every padding of the head dim
    split = {c[3] // c[4] for c in attention.ACTIVE if c[6] > 1}
    assert split >= {40, 64, 80, 104, 128, 160}, sorted(split)


def test_merges_of_the_gpu_cases(forms, tmp_path):
    """Every number of parts that a merge requests at once has a case at that many splits; what is requested covers the splits."""
    assert forms([c[:5] for c in attention.MERGES]) == [c[5:] for c in attention.MERGES]
    (tmp_path / "merge.cpp").write_text('#include <cstdio>\n#include "%s/attention_choice.h"\nint main() { for (int s = 2; s <= fise::AT_MAX_SPLITS; ++s) std::printf("%%d ", fise::at_merge(s)); }' % build.CSRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "merge"), str(tmp_path / "merge.cpp")], check=True)
    parts = dict(enumerate(map(int, subprocess.run([str(tmp_path / "merge")], check=True, capture_output=True, text=True).stdout.split()), 2))
    assert len(parts) == 31 and all(p >= s for s, p in parts.items())
    tested = {c[6] for c in attention.ACTIVE + attention.MERGES}
    assert set(parts.values()) <= tested, (set(parts.values()), tested)


def test_forms_of_the_partial_key_blocks(forms):
    """The kernel for many queries has a partial block at every head dim, as the first one and behind a whole one; so has the one for few."""
    def of(M, heads, d, N):
        return forms([(2, M, N, d * heads, heads)])[0][0]
    for d in attention.PARTIAL_D:
        for N in attention.PARTIAL_N:
            assert of(520, 8, d, N) == 1, (d, N)
        assert of(35, 2, d, 65) == 0 and of(35, 2, d, 120) == 0 and (d == 160 or of(35, 2, d, 9) == 0), d


def test_long_key_ranges_run_in_turns(tmp_path):
    """attention_turns_kernel has the cases of test_attention_long_key_ranges, in one part and in several, and nothing of other heads or of few key blocks."""
    (tmp_path / "turns.cpp").write_text('#include <cstdio>\n#include "%s/attention_choice.h"\nint main() { int M, n, d; while (std::scanf("%%d %%d %%d", &M, &n, &d) == 3) for (int ws = 0; ws < 2; ++ws) {'
                                        ' const int s = fise::attention_form(2, M, n, (n + 7) / 8 * 8, 8 * d, 8, ws); std::printf("%%d %%d\\n", s, fise::attention_turns(n, (n + 7) / 8 * 8, d, s)); } }' % build.CSRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "turns"), str(tmp_path / "turns.cpp")], check=True)

    def run(shapes):
        r = subprocess.run([str(tmp_path / "turns")], input="\n".join(f"{M} {N} {d}" for d, N, M in shapes), check=True, capture_output=True, text=True)
        return [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    forms = run(attention.TURNS)
    for d in (40, 80, 160):
        of = [f for t, pair in zip(attention.TURNS, zip(forms[::2], forms[1::2])) if t[0] == d for f in pair]
        assert (1, 1) in of and any(s > 1 and turns for s, turns in of), (d, of)
        for ends in (0, 1, 33, 63):                      # keys behind the last whole turn of 64
            assert any(N % 64 == ends and f == (1, 1) for (_, N, _), f in zip((t for t in attention.TURNS if t[0] == d for _ in (0, 1)), of)) or (d == 160 and ends == 63), (d, ends, of)
    assert run([(40, 705, 2000), (40, 704, 2000), (80, 705, 2000), (80, 704, 2000), (160, 449, 2000), (160, 448, 2000)])[::2] == [(1, 1), (1, 0)] * 3
    assert not any(turns for _, turns in run([(d, 447, 600) for d in (40, 80, 160)] + [(d, 2000, 600) for d in (32, 64, 104, 128, 152)]))


def test_forms_of_the_cross_attention(tmp_path):
    """One launch, two or three for a layer: the cases of test_gpu_cross.py have each at every width that has it, and 640 channels stop at one round of the CUs."""
    (tmp_path / "cross.cpp").write_text('#include <cstdio>\n#include "%s/attention_choice.h"\nint main() { int C, h, n, B, Ma, HW; while (std::scanf("%%d %%d %%d %%d %%d %%d", &C, &h, &n, &B, &Ma, &HW) == 6)'
                                        ' std::printf("%%d\\n", fise::cross_form(C, h, n, (n + 7) / 8 * 8, B, Ma, HW)); }' % build.CSRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "cross"), str(tmp_path / "cross.cpp")], check=True)

    def forms(shapes):                                   # (channels, heads, keys, batch, rows of an element, pixels)
        r = subprocess.run([str(tmp_path / "cross")], input="\n".join(" ".join(map(str, s)) for s in shapes), check=True, capture_output=True, text=True)
        return [int(v) for v in r.stdout.split()]
    cases = [c for p in cross.test_cross_attention_layer.pytestmark if p.name == "parametrize" for c in p.args[1]]
    got = forms([(C, 8, n, B, max(1, (H // t) * (W // t) - 3) * t * t, H * W) for C, B, H, W, t, n in cases])
    assert {(c[0], f) for c, f in zip(cases, got)} == {(320, 0), (320, 1), (320, 2), (640, 0), (640, 1)}
    assert all(f == 0 for c, f in zip(cases, got) if c[-1] > 80)
    assert forms([(640, 8, 77, 1, 1024, 4096), (640, 8, 77, 1, 1025, 4096), (640, 8, 77, 32, 9, 256), (640, 8, 77, 33, 9, 256), (640, 8, 77, 2, 1024, 4096)]) == [1, 0, 1, 0, 0]
    assert forms([(320, 8, 77, 1, 1248, 4096), (320, 8, 77, 1, 1249, 4096), (320, 4, 77, 1, 1249, 4096), (1280, 8, 77, 1, 32, 64)]) == [1, 2, 0, 0]
