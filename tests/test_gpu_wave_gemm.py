"""GPU parity of the wave-split gathered GEMM at the sizes where its tiles, K shares and splits can go wrong, against the oracle's
masked convolution."""
import math
import zlib

import numpy as np
import pytest
import torch

from oracle import fise_oracle as fo
from paper_2305_17423_amd import workloads as wl
from helpers import DEV, TOL, dev, host, idx_dev, active_mask, check_map

pytestmark = pytest.mark.gpu
DT = "bf16"


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


CASES = [
    # name, form, B, H(out), W(out), C0, C1, Cout, k, stride, ups, tile, tiles, temb, res.  Which form a case runs is the launcher's choice:
    # test_launch_forms.py asks it, and that every form has cases.
    ("one-row-one-step", "private 32x32", 1, 8, 8, 64, 0, 4, 1, 1, 0, 1, 1, False, False),              # three of four waves without work
    ("32-rows-exact", "private 32x32", 2, 8, 8, 64, 64, 32, 1, 1, 0, 4, 1, False, True),
    ("33-rows-ragged-columns", "private 32x32", 1, 8, 8, 192, 0, 68, 3, 1, 0, 1, 33, True, True),
    ("source-change-inside-a-share", "private 32x32", 2, 8, 8, 64, 128, 96, 3, 1, 0, 2, 5, False, False),
    ("uneven-shares", "private 32x32", 1, 8, 8, 320, 0, 64, 1, 1, 0, 2, 3, False, True),                # 5 steps: shares of 2, 2, 1, 0
    ("split-over-workgroups", "private 32x32 in 6", 2, 8, 8, 640, 0, 36, 3, 1, 0, 2, 2, True, True),
    ("split-stride-2", "private 32x32 in 8", 1, 8, 8, 320, 320, 64, 3, 2, 0, 4, 2, False, False),
    ("split-upsample", "private 32x32 in 8", 1, 16, 16, 640, 0, 64, 3, 1, 1, 4, 3, False, False),
    ("many-row-tiles-long-k", "private 32x32", 1, 32, 32, 320, 0, 64, 3, 1, 0, 4, 39, True, False),     # row tiles fetch the weight slice together
    # (the four names with "block" are those of cases that were made for a shared ring and run on rings per wave)
    ("block-one-step", "private 32x64", 2, 64, 40, 64, 0, 160, 1, 1, 0, 8, 16, False, False),
    ("block-ragged-rows", "private 32x64", 1, 64, 64, 64, 0, 160, 3, 1, 0, 4, 129, True, True),         # 2064 rows, 9 steps
    ("block-stride-2", "private 32x64", 1, 64, 40, 64, 0, 160, 3, 2, 0, 8, 33, False, False),
    ("block-upsample", "private 32x64", 1, 64, 40, 128, 0, 160, 3, 1, 1, 8, 33, False, True),
    ("32x64-split", "private 32x64 in 5", 1, 24, 24, 640, 320, 324, 3, 2, 0, 4, 15, True, True),        # 27 steps each, shares of 7, 7, 7, 6
    ("64x64-own-rings", "private 64x64", 1, 48, 40, 128, 64, 324, 3, 1, 1, 4, 105, True, True),         # 1680 rows: half a last tile
    ("64x64-own-rings-split", "private 64x64 in 5", 1, 24, 24, 640, 640, 324, 3, 1, 1, 4, 30, False, True),
    # one ring for the workgroup: one step (the second of the pair is zeros), even and odd numbers of them, every source change
    ("64-row-tiles", "ring 64x64", 2, 64, 32, 128, 0, 324, 1, 1, 0, 8, 31, False, True),
    ("ring-one-step", "ring 64x64", 1, 48, 48, 64, 0, 324, 1, 1, 0, 4, 89, True, True),                 # 1424 rows
    ("ring-stride-2", "ring 64x64", 1, 64, 64, 64, 128, 324, 3, 2, 0, 8, 57, True, False),              # 27 steps
    ("ring-upsample-long-k", "ring 64x64", 1, 64, 80, 320, 0, 324, 3, 1, 1, 8, 77, False, True),        # 45 steps: row tiles fetch the weight slice together
    ("ring-split", "ring 64x64 in 2", 1, 40, 40, 320, 0, 324, 3, 1, 1, 4, 89, True, True),              # shares of 23 and 22 steps
    # 64 x 160 tiles: ragged rows, source changes, odd numbers of steps, splits
    ("block-27-steps", "block 64x160", 2, 48, 48, 64, 128, 640, 3, 1, 1, 4, 127, True, True),           # 4064 rows: half a last tile
    ("block-27-steps-stride-2", "block 64x160", 1, 72, 64, 128, 64, 640, 3, 2, 0, 4, 253, False, True),
    ("block-long-k-split", "block 64x160 in 4", 1, 64, 56, 640, 320, 160, 3, 1, 1, 4, 207, True, True), # 3312 rows, shares of 34, 34, 34, 33 steps
    ("block-patches-would-fit", "block 64x160", 1, 48, 44, 64, 64, 1280, 3, 1, 0, 2, 481, True, True),
    # patches of the tiles and their rings in LDS: tiles at corners and edges, strips that are half a tile, row tiles with absent strips, ragged
    # columns, source changes, splits
    ("block-sources", "patch 64x64", 2, 64, 40, 64, 128, 320, 3, 1, 0, 8, 17, True, False),
    ("block-long-k", "patch 64x32", 2, 64, 40, 320, 0, 160, 3, 1, 0, 8, 19, False, True),
    ("block-split", "patch 64x32", 2, 32, 32, 640, 0, 320, 3, 1, 0, 4, 32, True, True),                 # 1024 rows
    ("block-ragged-columns", "patch 64x64", 1, 64, 64, 64, 0, 324, 3, 1, 0, 4, 131, True, True),
    ("block-160-wide", "patch 64x64", 1, 64, 64, 640, 640, 320, 3, 1, 0, 8, 33, True, False),
    ("patch8-32x32", "patch 32x32", 2, 32, 64, 320, 320, 324, 3, 1, 0, 8, 4, True, True),               # half tiles of four rows
    ("patch8-64x32", "patch 64x32", 2, 64, 40, 320, 0, 320, 3, 1, 0, 8, 7, True, True),
    ("patch8-64x64", "patch 64x64", 1, 64, 80, 256, 64, 320, 3, 1, 0, 8, 41, False, True),              # source change behind four chunks
    ("patch8-odd-tiles", "patch 64x32", 2, 40, 64, 192, 128, 320, 3, 1, 0, 8, 9, True, False),
    ("patch4-32x32", "patch 32x32", 2, 24, 40, 640, 0, 260, 3, 1, 0, 4, 19, True, True),
    ("patch4-64x32-tail", "patch 32x32", 1, 48, 32, 640, 64, 320, 3, 1, 0, 4, 45, False, True),         # 720 rows: one strip of two in the last row tile
    ("patch4-64x32-one-strip", "patch 64x32", 1, 48, 32, 640, 64, 320, 3, 1, 0, 4, 57, True, True),     # 912 rows: one strip of four in the last row tile
    ("patch4-64x64", "patch 64x64", 2, 48, 48, 320, 320, 640, 3, 1, 0, 4, 43, True, False),
    ("patch4-split", "patch 64x32 in 3", 2, 16, 40, 640, 640, 640, 3, 1, 0, 4, 7, True, True),
    ("patch4-32x32-split", "patch 32x32 in 4", 1, 16, 40, 1280, 1280, 324, 3, 1, 0, 4, 9, True, True),
    ("patch4-64x64-split", "patch 64x64 in 5", 1, 32, 32, 1280, 640, 324, 3, 1, 0, 4, 30, False, True),
    ("patch2-64x32-split", "patch 64x32 in 2", 2, 16, 16, 1280, 0, 1280, 3, 1, 0, 2, 21, False, True),
    ("patch2-64x64", "patch 64x64", 2, 24, 24, 640, 0, 640, 3, 1, 0, 2, 101, True, False),              # 808 rows: ten strips in the last row tile
    ("patch2-all-tiles", "patch 64x32", 1, 16, 24, 640, 64, 1280, 3, 1, 0, 2, 96, False, False),
    # 64 or 128 rows x 80 columns (conv_patch.hip): row tiles whose last strips are absent or belong to the next batch element, one chunk of channels and
    # odd and even numbers of them, source changes
    ("wide8-128-one-chunk-tail", "wide 128x80", 1, 96, 80, 64, 0, 320, 3, 1, 0, 8, 119, True, True),
    ("wide8-128-sources-two-batches", "wide 128x80", 2, 64, 64, 64, 64, 320, 3, 1, 0, 8, 59, True, False),
    ("wide8-128-three-chunks", "wide 128x80", 2, 64, 64, 64, 128, 320, 3, 1, 0, 8, 64, False, True),
    ("wide8-64", "wide 64x80", 1, 64, 64, 192, 0, 320, 3, 1, 0, 8, 57, True, True),
    ("wide8-64-narrow-map", "wide 64x80", 2, 32, 64, 64, 64, 640, 3, 1, 0, 8, 15, False, True),
    ("wide4-64-tail", "wide 64x80", 1, 48, 40, 64, 128, 640, 3, 1, 0, 4, 113, True, True),
    ("wide4-64-two-batches", "wide 64x80", 2, 40, 24, 128, 0, 1280, 3, 1, 0, 4, 31, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_wave_gemm_edges(fb, case):
    name, _, B, Ho, Wo, C0, C1, Co, k, stride, ups, t, n, use_temb, use_res = case
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    H, W = (Ho // 2, Wo // 2) if ups else (Ho * stride, Wo * stride)
    x0 = wl.normal(rng, (B, H, W, C0), 1.0, DT)
    x1 = wl.normal(rng, (B, H, W, C1), 1.0, DT) if C1 else None
    w = wl.normal(rng, (Co, k, k, C0 + C1), 1 / math.sqrt(k * k * (C0 + C1)), DT)
    bias = wl.normal(rng, (Co,), 0.1, DT)
    temb = wl.normal(rng, (B, Co), 0.3) if use_temb else None
    res = wl.normal(rng, (B, Ho, Wo, Co), 1.0, DT) if use_res else None
    cache = wl.normal(rng, (B, Ho, Wo, Co), 1.0, DT)
    ix = np.sort(rng.choice((Ho // t) * (Wo // t), n, replace=False)).astype(np.int32)
    want = fo.masked_conv([x0, x1] if C1 else x0, w, bias, ix, t, cache.astype(np.float64).copy(), DT, stride=stride, upsample=bool(ups),
                          temb=temb, residual=res)
    y, xd, x1d, wd, bd, ixd = dev(cache, DT), dev(x0, DT), dev(x1, DT) if C1 else None, dev(w, DT), dev(bias, DT), idx_dev(ix)
    tembd, resd = dev(temb) if use_temb else None, dev(res, DT) if use_res else None
    a = fb.conv_args(xd, wd, bd, ixd, n, t, y, x1=x1d, ksize=k, stride=stride, upsample=ups, temb=tembd, residual=resd)
    ws = torch.full((fb.fise_masked_conv_workspace_bytes(a),), 0xA5, dtype=torch.uint8, device=DEV)
    fb.fise_masked_conv(a, ws)
    got = host(y)
    check_map(got, want, cache.astype(np.float64), active_mask(ix, t, Ho, Wo), TOL[DT], name)
    fb.fise_masked_conv(a, ws)                       # arrival counters are back at zero, the sum does not depend on who came last
    assert np.array_equal(host(y), got)


@pytest.mark.parametrize("C", [320, 384])           # behind the LayerNorm in one launch; three sections of one launch on a ring
def test_block_tile_rows_and_transposed_columns(fb, C):
    """Compact rows in, rows / scattered rows / transposed columns out: an attention layer of more than 2048 queries."""
    B, H, W, heads, t = 2, 48, 56, 8, 4
    rng = np.random.default_rng(41)
    x = wl.normal(rng, (B, H, W, C), 1.0, DT)
    Kc, Vc = (wl.normal(rng, (B, H * W, C), 1.0, DT) for _ in range(2))
    Wq, Wk, Wv, Wo = (wl.normal(rng, (C, C), C ** -0.5, DT) for _ in range(4))
    bo, gamma, beta = wl.normal(rng, (C,), 0.1, DT), np.ones(C, np.float32), np.zeros(C, np.float32)
    y0 = wl.normal(rng, (B, H, W, C), 1.0, DT)
    ix = np.sort(rng.choice((H // t) * (W // t), 67, replace=False)).astype(np.int32)
    y, Kd, Vtd = dev(y0, DT), dev(Kc, DT), dev(np.ascontiguousarray(Vc.transpose(0, 2, 1)), DT)
    ws = torch.zeros(fb.fise_masked_attention_workspace_bytes(B, C, ix.size, t), dtype=torch.uint8, device=DEV)
    ws_args = [dev(v, DT) for v in (x, gamma, beta, Wq, Wk, Wv, Wo, bo)]
    fb.fise_masked_attention(*ws_args, heads, Kd, Vtd, None, None, 0, idx_dev(ix), ix.size, t, y, ws)
    act = active_mask(ix, t, H, W)
    n = np.asarray(x, np.float64)[:, act]                     # [B, active, C]; rows normalised in float64, rounded once
    n = (n - n.mean(-1, keepdims=True)) / np.sqrt(n.var(-1, keepdims=True) + 1e-5)
    for got, w, cache in ((host(Kd), Wk, Kc), (host(Vtd).transpose(0, 2, 1), Wv, Vc)):
        got, cache = got.reshape(B, H, W, C), np.asarray(cache, np.float64).reshape(B, H, W, C)
        want = cache.copy()
        want[:, act] = n @ np.asarray(w, np.float64).T
        check_map(got, want, cache, act, TOL[DT], "keys or values")
    K64, V64 = host(Kd).astype(np.float64), host(Vtd).astype(np.float64).transpose(0, 2, 1)
    q, d, o = n @ np.asarray(Wq, np.float64).T, C // heads, []
    for h in range(heads):
        c = slice(h * d, (h + 1) * d)
        s = q[..., c] @ K64[..., c].transpose(0, 2, 1) / math.sqrt(d)
        p = np.exp(s - s.max(-1, keepdims=True))
        o.append(p @ V64[..., c] / p.sum(-1, keepdims=True))
    want = np.asarray(y0, np.float64).copy()
    want[:, act] = np.concatenate(o, -1) @ np.asarray(Wo, np.float64).T + np.asarray(bo, np.float64) + np.asarray(x, np.float64)[:, act]
    check_map(host(y), want, np.asarray(y0, np.float64), act, TOL[DT], "layer output")


# (the last size one by one; test_launch_forms.py has the tiles of the others)
PRODUCTS = [(1, 1, 64, 64), (2, 77, 768, 320), (1, 100, 256, 1280), (1, 8, 768, 1280), (4, 154, 768, 640), (2, 33, 128, 192), (4, 77, 768, 1280), (4, 154, 192, 1280),
            (2, 77, 96, 320)]


@pytest.mark.parametrize("B,n,Dc,C", PRODUCTS)
def test_products_of_one_launch(fb, B, n, Dc, C):
    """Keys and values of a context: two products of the same rows, rows out and transposed columns out."""
    rng = np.random.default_rng(B * 1000 + n)
    ctx, wk, wv = wl.normal(rng, (B, n, Dc), 1.0, DT), wl.normal(rng, (C, Dc), Dc ** -0.5, DT), wl.normal(rng, (C, Dc), Dc ** -0.5, DT)
    stride = (n + 7) // 8 * 8
    K = torch.full((B, n, C), 7.0, dtype=torch.bfloat16, device=DEV)
    Vt = torch.full((B, C, stride), 7.0, dtype=torch.bfloat16, device=DEV)
    fb.fise_context_kv(dev(ctx, DT), dev(wk, DT), dev(wv, DT), K, Vt)
    for got, w in ((host(K), wk), (host(Vt)[:, :, :n].transpose(0, 2, 1), wv)):
        want = np.asarray(ctx, np.float64) @ np.asarray(w, np.float64).T
        assert np.abs(got - want).max() <= TOL[DT] * max(1.0, np.sqrt((want ** 2).mean()))
    assert (host(Vt)[:, :, n:] == 7.0).all()         # columns past the context stay as they are
