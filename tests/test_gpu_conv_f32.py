"""GPU parity of the fp32 convolution of a few tiles (K range shared by the waves of a workgroup) at the edges of its tiles, of its
batches of K units and of the rule that chooses it, against the oracle's masked convolution."""
import math
import zlib

import numpy as np
import pytest
import torch

from oracle import fise_oracle as fo
from paper_2305_17423_amd import workloads as wl
from helpers import DEV, dev, host, idx_dev, active_mask, check_map

pytestmark = pytest.mark.gpu
CASES = [
    # name, B, H(out), W(out), Cin, Cout, k, stride, ups, tile, tiles, temb, res
    ("one-row-two-units", 1, 8, 8, 16, 4, 1, 1, 0, 1, 1, False, False),               # six of eight waves without work
    ("33-rows-ragged-columns", 1, 8, 8, 48, 36, 3, 1, 0, 1, 33, True, True),           # 54 units: batches end inside
    ("border-tiles", 2, 8, 8, 64, 64, 3, 1, 0, 4, 4, False, True),                     # 72 units: one batch of nine for each of eight waves
    ("a-batch-and-a-unit", 1, 8, 8, 592, 40, 1, 1, 0, 2, 9, True, False),              # 74 units: two waves take a tenth
    ("stride-2", 2, 8, 8, 128, 32, 3, 2, 0, 2, 5, True, False),
    ("upsample", 1, 16, 16, 32, 68, 3, 1, 1, 4, 7, False, False),
    ("256-tiles", 2, 64, 32, 16, 64, 3, 1, 0, 8, 32, False, False),                    # 128 x 2 tiles: the last launch shape of this kernel
    ("258-tiles", 1, 64, 72, 16, 36, 3, 1, 0, 4, 258, False, True),                    # the staged kernel, 16 channels of a tap at a time
    ("258-tiles-32-channels", 1, 64, 72, 32, 36, 3, 1, 0, 4, 258, True, False),        # and 32
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_conv_f32_few_tiles(case):
    from paper_2305_17423_amd import binding as fb
    name, B, Ho, Wo, Ci, Co, k, stride, ups, t, n, use_temb, use_res = case
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    H, W = (Ho // 2, Wo // 2) if ups else (Ho * stride, Wo * stride)
    x = wl.normal(rng, (B, H, W, Ci), 1.0)
    w = wl.normal(rng, (Co, k, k, Ci), 1 / math.sqrt(k * k * Ci))
    bias = wl.normal(rng, (Co,), 0.1)
    temb = wl.normal(rng, (B, Co), 0.3) if use_temb else None
    res = wl.normal(rng, (B, Ho, Wo, Co), 1.0) if use_res else None
    cache = wl.normal(rng, (B, Ho, Wo, Co), 1.0)
    ix = np.sort(rng.choice((Ho // t) * (Wo // t), n, replace=False)).astype(np.int32)
    want = fo.masked_conv(x, w, bias, ix, t, cache.astype(np.float64).copy(), "f32", stride=stride, upsample=bool(ups), temb=temb, residual=res)
    y, xd, wd, bd, ixd = dev(cache), dev(x), dev(w), dev(bias), idx_dev(ix)
    tembd, resd = dev(temb) if use_temb else None, dev(res) if use_res else None
    fb.fise_masked_conv(fb.conv_args(xd, wd, bd, ixd, n, t, y, ksize=k, stride=stride, upsample=ups, temb=tembd, residual=resd), None)
    # K <= 1152 float products and sums: K 2^-24 = 7e-5 of the largest term at worst, 1e-5 as the sums here go
    check_map(host(y), want, cache.astype(np.float64), active_mask(ix, t, Ho, Wo), 1e-5, name)


FORMS = [
    # tiles of 16 x 16 up to 512 of them, 32 x 32 up to 256 of those: both sides of the rule, rows and columns that end inside a tile, batches that end inside
    ("16-row-tiles-17-rows", 1, 8, 8, 80, 20, 3, 1, 0, 1, 17, True, True),                # 45 units of 16 channels: two batches of five for five of eight waves
    ("16-row-tiles-512", 1, 64, 64, 32, 32, 3, 1, 0, 8, 64, False, True),
    ("32-row-tiles-4001-rows", 1, 64, 64, 48, 36, 3, 1, 0, 1, 4001, True, True),          # 252 tiles of 32 x 32
    ("32-row-tiles-a-batch-and-a-unit", 1, 64, 64, 592, 68, 1, 1, 0, 1, 2700, True, False),
    ("32-row-tiles-stride-2", 2, 64, 32, 32, 64, 3, 2, 0, 8, 32, False, True),
]


@pytest.mark.parametrize("case", FORMS, ids=[c[0] for c in FORMS])
def test_conv_f32_forms_of_the_wave_kernel(case):
    test_conv_f32_few_tiles(case)


@pytest.mark.parametrize("C,co,tiles", [(64, 64, 16), (320, 64, 4), (1280, 64, 1), (320, 68, 3)])
def test_conv_f32_of_few_tiles_is_as_close_to_64_bits_as_its_chains_of_additions(C, co, tiles):
    """Tiles of 16 x 16: eight waves of four accumulators share K, so a chain is K / 32 additions, whose roundings of 2^-24 / sqrt(3) in the mean leave
    sqrt(K / 64) of them, and the 32 sums about five.  A chain of K / 8 is over it."""
    from paper_2305_17423_amd import binding as fb
    B, H, W, t = 1, 32, 32, 4
    g = torch.Generator(device=DEV).manual_seed(C)
    x, w = torch.randn(B, H, W, C, generator=g, device=DEV), torch.randn(co, 3, 3, C, generator=g, device=DEV) * (9 * C) ** -0.5
    idx = torch.randperm((H // t) * (W // t), generator=g, device=DEV)[:tiles].sort().values.to(torch.int32)
    active = torch.zeros((H // t) * (W // t), dtype=torch.bool, device=DEV)
    active[idx.long()] = True
    active = active.reshape(H // t, W // t).repeat_interleave(t, 0).repeat_interleave(t, 1).cpu()
    y = torch.zeros(B, H, W, co, device=DEV)
    fb.fise_masked_conv(fb.conv_args(x, w, None, idx, tiles, t, y), None)
    want = torch.nn.functional.conv2d(x.cpu().double().permute(0, 3, 1, 2), w.cpu().double().permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)[:, active]
    err = float((y.cpu().double()[:, active] - want).norm() / want.norm())
    assert err <= 2.0 ** -24 / 3 ** 0.5 * (9 * C / 64 + 5) ** 0.5, err
