"""GPU parity of the cross-attention layer over map pixels where its forms of few launches end: key counts around its tiles of 16 and 32 keys and past the last
one, row tiles that end inside a batch element, tiles whose pixels are no runs of four, one batch element and three, few rows and many (one launch for the layer
from forty workgroups of 32 rows on, below and at 640 channels a workgroup per head and the product behind it).  The float rows of a transformer block
have their cases in test_gpu_blocks.py."""
import pytest
import torch

from helpers import DEV

pytestmark = pytest.mark.gpu


MANY = [(2, 64, 64, 8, 77), (2, 36, 36, 3, 77), (1, 36, 40, 4, 1), (3, 24, 20, 2, 8), (2, 28, 26, 1, 31), (1, 64, 40, 8, 32), (2, 28, 28, 4, 33), (2, 32, 24, 4, 48), (1, 48, 32, 4, 63),
        (2, 28, 28, 4, 64), (2, 28, 28, 4, 65), (2, 28, 28, 4, 72), (2, 28, 28, 4, 80), (2, 28, 28, 4, 81)]
FEW = [(1, 8, 8, 1, 77), (2, 12, 12, 3, 77), (1, 20, 16, 4, 1), (3, 10, 10, 2, 8), (2, 12, 8, 4, 31), (2, 16, 16, 4, 33), (1, 32, 24, 8, 63), (2, 12, 12, 2, 64), (2, 12, 12, 4, 65), (2, 12, 20, 4, 80), (1, 12, 12, 4, 81)]


@pytest.mark.parametrize("C,B,H,W,tile,n_ctx", [(320, *c) for c in MANY + FEW] + [(640, *c) for c in FEW + MANY[:3]])
def test_cross_attention_layer(C, B, H, W, tile, n_ctx):
    from paper_2305_17423_amd import binding as fb
    heads, stride = 8, (n_ctx + 7) // 8 * 8 + 8
    g = torch.Generator(device=DEV).manual_seed(n_ctx + H)
    normal = lambda *shape, std=1.0: (torch.randn(*shape, generator=g, device=DEV) * std).bfloat16()      # noqa: E731
    x, y = normal(B, H, W, C), normal(B, H, W, C)
    gam, bet, wq, wo, bo = 1 + normal(C, std=0.1), normal(C, std=0.1), normal(C, C, std=1.4 * C ** -0.5), normal(C, C, std=0.9 * C ** -0.5), normal(C, std=0.1)
    K, V = normal(B, n_ctx, C), torch.full((B, C, stride), float("nan"), dtype=torch.bfloat16, device=DEV)      # the columns past the last key hold anything
    V[:, :, :n_ctx] = normal(B, C, n_ctx)
    tiles = (H // tile) * (W // tile)
    idx = torch.randperm(tiles, generator=g, device=DEV)[: max(1, tiles - 3)].sort().values.to(torch.int32)
    active = torch.zeros(tiles, dtype=torch.bool, device=DEV)
    active[idx.long()] = True
    active = active.reshape(H // tile, W // tile).repeat_interleave(tile, 0).repeat_interleave(tile, 1)
    before = y.clone()
    ws = torch.zeros(int(fb.fise_masked_attention_workspace_bytes(B, C, idx.numel(), tile)), dtype=torch.uint8, device=DEV)
    fb.fise_masked_attention(x, gam, bet, wq, None, None, wo, bo, heads, None, None, K, V, n_ctx, idx, idx.numel(), tile, y, ws)
    f = lambda t: t.float().cpu().double()                                                               # noqa: E731
    ln = torch.nn.functional.layer_norm(f(x).reshape(B, H * W, C), (C,), f(gam), f(bet), 1e-5)
    q = (ln @ f(wq).t()).reshape(B, -1, heads, C // heads).transpose(1, 2).contiguous()
    k = f(K).reshape(B, n_ctx, heads, -1).permute(0, 2, 3, 1).contiguous()
    v = f(V[:, :, :n_ctx]).reshape(B, heads, -1, n_ctx).transpose(2, 3).contiguous()
    o = ((q @ k) * (C // heads) ** -0.5).softmax(-1) @ v
    update = o.transpose(1, 2).reshape(B, H * W, C) @ f(wo).t() + f(bo)
    want = (f(x).reshape(B, H * W, C) + update).reshape(B, H, W, C)
    err = (f(y) - want)[:, active.cpu()]
    # the sum is stored in bf16 (2^-9 relative); normalised rows, queries, probabilities and outputs are rounded to bf16 on the way: 2^-8 of the update, twice
    rms = float(update.pow(2).mean().sqrt())
    assert bool((err.abs() <= want[:, active.cpu()].abs() * 2.0 ** -8 + rms * 0.1).all())
    assert float(err.pow(2).mean().sqrt()) <= 2.0 ** -9 * float(want.pow(2).mean().sqrt()) + rms * 2.0 ** -7
    assert torch.equal(y[:, ~active], before[:, ~active])


@pytest.mark.parametrize("key", [0, 31, 32, 70, 76])
@pytest.mark.parametrize("C,B,H,W,tile", [(320, 2, 16, 16, 4), (320, 2, 32, 32, 4), (640, 2, 16, 16, 4)])
def test_cross_attention_infinite_value(C, B, H, W, tile, key):
    """Every key has a weight, so an infinite value makes its channel infinite in every row, and the product every channel by the sign of its weight."""
    from paper_2305_17423_amd import binding as fb
    n_ctx, channel = 77, C // 2 + 5
    g = torch.Generator(device=DEV).manual_seed(key)
    normal = lambda *shape, std=1.0: (torch.randn(*shape, generator=g, device=DEV) * std).bfloat16()      # noqa: E731
    x, y = normal(B, H, W, C), normal(B, H, W, C)
    gam, bet, wq, wo = 1 + normal(C, std=0.1), normal(C, std=0.1), normal(C, C, std=C ** -0.5), normal(C, C, std=C ** -0.5)
    wo[:, channel] = torch.where(wo[:, channel] < 0, -1, 1)
    K, V = normal(B, n_ctx, C), torch.zeros((B, C, 80), dtype=torch.bfloat16, device=DEV)
    V[:, :, :n_ctx] = normal(B, C, n_ctx)
    V[:, channel, key] = float("inf")
    tiles = (H // tile) * (W // tile)
    idx = torch.arange(tiles, dtype=torch.int32, device=DEV)
    ws = torch.zeros(int(fb.fise_masked_attention_workspace_bytes(B, C, tiles, tile)), dtype=torch.uint8, device=DEV)
    fb.fise_masked_attention(x, gam, bet, wq, None, None, wo, None, 8, None, None, K, V, n_ctx, idx, tiles, tile, y, ws)
    assert torch.equal(y, (wo[:, channel] * float("inf")).expand_as(y))
