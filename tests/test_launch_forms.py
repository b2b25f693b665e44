"""Which kernel and tile the cases of the GPU tests run on: the launchers' own rules (csrc/gemm_choice.h), compiled for the host and asked with the
sizes of those cases.  A case that was made for a form and no longer runs it fails here, and so does a form that has lost its last case."""
import os
import subprocess

import pytest

import test_gpu_blocks as blocks
import test_gpu_conv as bf16
import test_gpu_conv_f32 as f32
import test_gpu_fresh_stats as fresh
import test_gpu_rows_group as group
import test_gpu_wave_gemm as gemm
from paper_2305_17423_amd import build

PROGRAM = r"""
#include <cstdio>
#include "%s/conv_choice.h"
#include "%s/gemm_choice.h"
using namespace fise;
int main() {
    const char* kinds[] = {"private", "ring", "block", "patch", "wide"};
    int what, v[9];
    while (std::scanf("%%d %%d %%d", &what, &v[0], &v[1]) == 3) {       // 0 rows N: a linear of many rows
        if (what == 0) { std::printf("%%d\n", 32 * linear_tile(v[0], v[1])); continue; }
        if (what == 2) {                                 // 2 B rows K N geglu gn: a product behind a normalisation, rows of a batch element
            for (int i = 2; i < 6; ++i) if (std::scanf("%%d", &v[i]) != 1) return 1;
            const NormChoice c = choose_norm_tile({v[0], v[1], v[2], v[3], v[4] != 0, v[5] != 0});
            if (c.tile < 0) { std::puts("none"); continue; }
            const NormTile& t = kNormTiles[c.tile];
            std::printf("%%d%%s %%dx%%d%%s\n", t.K, t.geglu ? " gated" : "", 16 * t.rt, 16 * t.ct, waves_per_unit(v[2] / 320, t.ct, c.per) ? " in parts" : "");
            continue;
        }
        if (what == 3) {                                 // 3 rows columns fours: a group of products
            if (std::scanf("%%d", &v[2]) != 1) return 1;
            std::printf("%%d\n", 32 * group_tile(v[0], v[1], v[2] != 0));
            continue;
        }
        if (what == 4) { std::printf("%%d\n", conv_f32_edge(v[0], v[1], 1 << 20)); continue; }       // 4 rows N: an fp32 convolution
        if (what == 5) {                                 // 5 C0 C1 N k stride upsample groupnorm adds tile tile_w n: is it four columns behind a GroupNorm
            int w[9];
            for (int& x : w) if (std::scanf("%%d", &x) != 1) return 1;
            std::printf("%%d\n", conv_out_takes({v[0], v[1], w[0], w[1], w[2], w[6], w[7], w[8], w[3] != 0, w[4] != 0, w[5] != 0}));
            continue;
        }
        if (what == 6) {                                 // 6 B pixels C G: pieces of eight channels that a lane holds for fresh statistics
            for (int i = 2; i < 4; ++i) if (std::scanf("%%d", &v[i]) != 1) return 1;
            std::printf("%%d\n", gn_map_values(gn_slab(v[2], v[3]), v[0], v[1], v[2], v[3]));
            continue;
        }
        for (int i = 2; i < 9; ++i) if (std::scanf("%%d", &v[i]) != 1) return 1;     // 1 rows N K K2 tile geglu patches one_map scratch
        const GemmShape g{v[0], v[1], v[2], v[3], v[4], v[5] != 0, v[6] != 0, v[7] != 0};
        const TileChoice c = choose_tile(g, v[8] ? IGEMM_PARTIAL_BYTES : 0);
        std::printf("%%s %%dx%%d", kinds[c.kind], 32 * c.tm, c.kind == WIDE ? 80 : 32 * c.tn);
        if (c.splits > 1) std::printf(" in %%d", c.splits);
        std::puts("");
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "forms.cpp").write_text(PROGRAM % (build.CSRC, build.CSRC))
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(d / "forms"), str(d / "forms.cpp")], check=True)

    def run(questions):
        r = subprocess.run([str(d / "forms")], input="\n".join(" ".join(str(int(v)) for v in q) for q in questions), check=True, capture_output=True, text=True)
        return r.stdout.splitlines()
    return run


def conv(rows, N, K, K2, k, stride, ups, tile):
    return 1, rows, N, K, K2, tile, 0, k == 3 and stride == 1 and not ups and tile in (2, 4, 8), 1, 1


def rows_gemm(rows, N, K, geglu=0, scratch=1):
    return 1, rows, N, K, 0, 4, geglu, 0, 0, scratch


def test_convolution_cases(ask):
    cases = gemm.CASES
    got = ask([conv(B * n * t * t, Co, k * k * (C0 + C1), 0, k, stride, ups, t) for _, _, B, _, _, C0, C1, Co, k, stride, ups, t, n, _, _ in cases])
    assert {c[0]: f for c, f in zip(cases, got)} == {c[0]: c[1] for c in cases}
    for name, _, _, Ho, Wo, *_, t, n, _, _ in cases:
        assert n <= (Ho // t) * (Wo // t), name
    forms = {c[1].split(" in ")[0] + (" in" if " in " in c[1] else "") for c in cases}
    assert forms == {"private 32x32", "private 32x32 in", "private 32x64", "private 32x64 in", "private 64x64", "private 64x64 in", "ring 64x64", "ring 64x64 in",
                     "block 64x160", "block 64x160 in", "patch 32x32", "patch 32x32 in", "patch 64x32", "patch 64x32 in", "patch 64x64", "patch 64x64 in",
                     "wide 64x80", "wide 128x80"}
    for edge, tiles in ((2, {"64x32", "64x64"}), (4, {"32x32", "64x32", "64x64"}), (8, {"32x32", "64x32", "64x64"})):
        assert {c[1].split()[1] for c in cases if c[1].startswith("patch") and c[11] == edge} == tiles
    assert {c[11] for c in cases if c[1] == "wide 64x80"} == {4, 8}


def test_product_group_cases(ask):
    """Without scratch; the last one is no multiple of 64 deep and runs product by product."""
    got = ask([rows_gemm(B * n, 2 * C, Dc, scratch=0) for B, n, Dc, C in gemm.PRODUCTS[:-1]])
    assert set(got) == {"private 32x32", "private 32x64", "private 64x64", "ring 64x64"}, got
    assert gemm.PRODUCTS[-1][2] % 64


def test_shortcut_cases(ask):
    for case in blocks.RES_CASES:
        name, B, H, W, C0, C1, Co, t, *_ = case
        if not name.startswith("wide"):
            continue
        rows = B * blocks.res_inputs(case)[5].size * t * t
        want = "wide %sx80" % name.split("-")[1]
        assert ask([conv(rows, Co, 9 * (C0 + C1), 0, 3, 1, 0, t), conv(rows, Co, 9 * Co, C0 + C1, 3, 1, 0, t)]) == [want, want], name


LINEARS = {"rows-2124-320": (2124, 64), "rows-2048-640": (2048, 64), "rows-4230-320": (4230, 128), "rows-2368-640": (2368, 128), "rows-1854-320": (1854, 0)}
GENERAL = {"general-192": (608, "private 32x64", "private 64x64"), "general-384": (1088, "ring 64x64", "ring 64x64")}      # rows, QKV, gated product


def test_transformer_cases(ask):
    seen = set()
    for case in blocks.TR_CASES:
        name, H, W, C, t, _ = case
        if name not in LINEARS and name not in GENERAL:
            continue
        rows = 2 * blocks.tr_inputs(case, blocks.tr_rng(case))[3].size * t * t
        if name in LINEARS:
            assert (rows, int(ask([(0, rows, C)])[0])) == LINEARS[name], name
        else:
            assert (rows, *ask([rows_gemm(rows, 3 * C, C), rows_gemm(rows, 4 * C, C, geglu=1)])) == GENERAL[name], name
        seen.add(name)
    assert seen == set(LINEARS) | set(GENERAL)


def norm_products(B, Ma, C):
    """1x1 in, query product, queries + keys + values, gated product of a block."""
    first = [(2, B, Ma, C, C, 0, 1)] if B == 1 or Ma >= (16 if C == 1280 else 32) else []      # fewer rows: another kernel
    return first + [(2, B, Ma, C, C, 0, 0), (2, B, Ma, C, 3 * C, 0, 0), (2, B, Ma, C, 4 * C, 1, 0)]


def test_products_behind_a_normalisation(ask):
    """Every tile, with K dealt out among the waves and without, that any number of rows reaches is one that a transformer block of the GPU tests runs."""
    rows = sorted({int(1.02 ** i) for i in range(462)})                                        # 1 to 9200
    reached = set(ask([q for C in (320, 640, 1280) for B in (1, 2, 4) for Ma in rows for q in norm_products(B, Ma, C)]))
    tested = set()
    for case in blocks.TR_CASES:
        if case[3] in (320, 640, 1280):
            tested |= set(ask(norm_products(2, blocks.tr_inputs(case, blocks.tr_rng(case))[3].size * case[4] ** 2, case[3])))
    assert len(reached) >= 19 and tested == reached, (reached - tested, tested - reached)


def test_groups_over_many_columns(ask):
    """Every row tile has a case; where a second or further round would be the slower form, the smaller tiles have the launch."""
    cases = [c for p in group.test_context_keys_and_values_of_many_layers.pytestmark if p.name == "parametrize" for c in p.args[1]]
    columns = 11 * 2 * 1280                              # of its eleven layers
    got = ask([(3, B * n, columns, n % 4 == 0) for B, n, _ in cases])
    assert set(got) >= {"32", "64", "96", "160", "224"}, got
    sd15 = 2 * (5 * 320 + 5 * 640 + 6 * 1280)
    rows = {(154, 0): 160, (224, 1): 224, (226, 0): 160, (240, 1): 0, (256, 1): 0, (264, 1): 160, (448, 1): 224, (512, 1): 0, (520, 0): 224, (576, 1): 0, (616, 0): 224, (896, 1): 224}
    assert ask([(3, r, sd15, f) for r, f in rows]) == [str(t) for t in rows.values()]
    assert ask([(3, 154, 17808, 0), (3, 154, 17824, 0)]) == ["0", "160"]


def test_fp32_convolution_cases(ask):
    """Tiles of 16 x 16 and of 32 x 32, both sides of the lines between them and behind them."""
    got = dict(zip((c[0] for c in f32.CASES + f32.FORMS), ask([(4, c[1] * c[10] * c[9] ** 2, c[5]) for c in f32.CASES + f32.FORMS])))
    assert set(got.values()) == {"16", "32", "0"} and all(got[c[0]] == c[0].split("-")[0] for c in f32.FORMS), got
    assert ask([(4, 512, 256), (4, 513, 256), (4, 4096, 64), (4, 4097, 64)]) == ["16", "32", "32", "0"]


def test_four_column_cases(ask):
    def question(case):
        name, B, H, W, C0, C1, Co, k, stride, ups, t, use_gn, silu, use_temb, use_res, frac = case
        th, tw = t if isinstance(t, tuple) else (t, t)
        return 5, C0, C1, Co, k, stride, ups, use_gn, use_temb or use_res, th, tw, 4
    assert ask([question(c) for c in bf16.NARROW]) == ["1"] * (len(bf16.NARROW) - 1) + ["0"]      # the last one is a width past the last
    taken = [c[0] for c, f in zip(bf16.CASES, ask([question(c) for c in bf16.CASES])) if f == "1"]
    assert taken == ["narrow-out"]                       # and nothing of other widths, strides, sources or additions
    assert ask([(5, 320, 0, 4, 3, 1, 0, 1, 0, 8, 8, 1 << 22), (5, 320, 0, 4, 3, 1, 0, 1, 0, 8, 4, 4), (5, 320, 0, 4, 3, 1, 0, 1, 0, 2, 2, 4)]) == ["0", "0", "0"]


def test_fresh_statistics_cases(ask):
    """A lane's four registers' worth of pieces, its eight, and maps too large for one launch."""
    cases = [c for p in fresh.test_resnet_block_with_fresh_statistics_of_an_active_map.pytestmark if p.name == "parametrize" for c in p.args[1]]
    for B, H, W, C, G, tile, tiles in cases:
        assert tiles * tile * tile == H * W
    got = [int(v) for v in ask([(6, B, H * W, C, G) for B, H, W, C, G, *_ in cases])]
    assert got[-2:] == [0, 0] and min(got[:-2]) == 1 and {1, 2, 3, 4} & set(got) and 8 in got, got
    assert ask([(6, 2, 64, 320, 40), (6, 1, 64, 256, 32), (6, 1, 64, 256, 16), (6, 2, 64, 96, 24), (6, 2, 64, 4104, 27), (6, 1, 4, 1 << 27, 1 << 15)]) == ["1", "1", "0", "0", "0", "0"]
