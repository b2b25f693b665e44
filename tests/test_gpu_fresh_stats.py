"""Fresh statistics worked out by the launch that applies them: group counts that are no powers of two, groups narrower than eight channels, one
and many chunks of pixels, a few active tiles; the statistics are those of the whole maps in 64 bits, the output that of the oracle."""
import numpy as np
import pytest
import torch

from oracle import fise_oracle as fo
from oracle import fise_unet_oracle as uo
from paper_2305_17423_amd import workloads as wl
from helpers import DEV, TOL, dev, host, idx_dev, active_mask, check_map
from test_gpu_blocks import res_shapes

pytestmark = pytest.mark.gpu
DT = "bf16"


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


@pytest.mark.parametrize("B,H,W,C,G,tile,tiles", [(1, 8, 8, 96, 24, 4, 1), (2, 24, 40, 96, 6, 4, 9), (2, 64, 72, 64, 64, 8, 3), (3, 16, 16, 160, 5, 2, 64),
                                                  # the most groups that the one launch holds, and more: statistics, then activation
                                                  (1, 8, 16, 512, 256, 4, 5), (2, 16, 16, 576, 288, 4, 9)])
def test_resnet_block_with_fresh_statistics(fb, B, H, W, C, G, tile, tiles):
    rng = np.random.default_rng(C + G + H)
    P = wl.params_from_shapes(rng, res_shapes("r", C, C, 64), 0.05, DT)
    x, h_old, out_old = (wl.normal(rng, (B, H, W, C), 1.0, DT) for _ in range(3))
    idx = np.sort(rng.choice((H // tile) * (W // tile), tiles, replace=False)).astype(np.int32)
    emb = wl.normal(rng, (B, 64), 1.0)
    want = {"r.h1": h_old.astype(np.float64), "r.out": out_old.astype(np.float64)}
    uo.resnet_block(P, "r", x, emb, want, idx, tile, DT, G, stats="fresh")
    tproj = fo.linear(uo._silu(emb.astype(np.float64)), P["r.temb.w"], P["r.temb.b"])
    keep = []
    h1, out = dev(h_old, DT), dev(out_old, DT)
    m1, r1, m2, r2 = (torch.zeros((B, G), device=DEV) for _ in range(4))
    d = lambda k: dev(P["r." + k], DT)
    a = fb.fill_args(fb.fise_resnet_args, keep, x0=dev(x, DT), x1=None, C0=C, C1=0, B=B, H=H, W=W, Cout=C, G=G, gn1_mean=m1, gn1_rstd=r1,
                     gn1_gamma=d("gn1.g"), gn1_beta=d("gn1.b"), conv1_w=d("conv1.w"), conv1_b=d("conv1.b"), temb=dev(tproj), temb_stride=C,
                     gn2_mean=m2, gn2_rstd=r2, gn2_gamma=d("gn2.g"), gn2_beta=d("gn2.b"), conv2_w=d("conv2.w"), conv2_b=d("conv2.b"),
                     sc_w=None, sc_b=None, tile_idx=idx_dev(idx), n_active=idx.size, tile=tile, h1_cache=h1, out_cache=out, stats_fresh=1)
    ws = torch.full((max(fb.fise_masked_resnet_block_workspace_bytes(a), 256),), 0x7F, dtype=torch.uint8, device=DEV)
    fb.fise_masked_resnet_block(a, ws)
    for v, mean, rstd in ((x, m1, r1), (host(h1), m2, r2)):      # the second ones are those of the map the first convolution left
        g = np.asarray(v, np.float64).reshape(B, H * W, G, C // G)
        m, var = g.mean((1, 3)), g.var((1, 3))
        # 64-bit sums of float sums of a few dozen terms each, stored as floats
        assert np.abs(host(mean) - m).max() < 2e-6 and np.abs(host(rstd) * np.sqrt(var + 1e-5) - 1).max() < 2e-6
    act = active_mask(idx, tile, H, W)
    check_map(host(h1), want["r.h1"], h_old, act, TOL[DT], "h1")
    check_map(host(out), want["r.out"], out_old, act, TOL[DT], "out")


# every pixel of a small map active: pieces of 8 channels inside a group and across its edge, 1 to 8 pieces a lane, pixels that leave lanes idle,
# three batch elements; the last two are maps that are too large for one launch
@pytest.mark.parametrize("B,H,W,C,G,tile,tiles", [(2, 16, 16, 256, 32, 4, 16), (2, 8, 8, 640, 32, 2, 16), (3, 16, 24, 384, 32, 8, 6), (2, 24, 24, 640, 32, 8, 9),
                                                  (8, 16, 24, 288, 32, 8, 6), (2, 24, 34, 640, 32, 2, 204), (2, 28, 32, 640, 32, 4, 56), (8, 24, 24, 288, 32, 8, 9)])
def test_resnet_block_with_fresh_statistics_of_an_active_map(fb, B, H, W, C, G, tile, tiles):
    test_resnet_block_with_fresh_statistics(fb, B, H, W, C, G, tile, tiles)
