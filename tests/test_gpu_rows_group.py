"""GPU parity of the products of a group of cross-attention layers (keys and transposed values of a prompt) where their tiles end: rows around the row
tiles of a workgroup, column tiles that end one product and begin the next, fewer stages of K than the ring holds."""
import pytest
import torch

from helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_ctx,ctx_dim", [(1, 1, 64), (1, 32, 128), (1, 33, 768), (2, 32, 192), (1, 65, 64), (4, 24, 320), (1, 97, 128), (2, 77, 768), (4, 40, 64),
                                             (1, 161, 768), (4, 56, 128), (1, 225, 64), (3, 107, 192), (4, 154, 768)])
def test_context_keys_and_values_of_many_layers(B, n_ctx, ctx_dim):
    from paper_2305_17423_amd import binding as fb
    d = dict(in_ch=4, out_ch=4, base=320, mults=(4, 4), layers=2, attn=(True, True), heads=8, ctx_dim=ctx_dim, n_ctx=n_ctx, groups=32, H=16, W=16, B=B)
    u = fb.fise_unet_create(d)
    try:
        g = torch.Generator(device=DEV).manual_seed(n_ctx)
        weights = torch.empty(fb.fise_unet_weight_elems(u), dtype=torch.bfloat16, device=DEV)        # only the layers' own are read
        where = {name: (off, num) for name, off, num in fb.fise_unet_tensors(u, 0)}
        ctx = torch.randn(B, n_ctx, ctx_dim, generator=g, device=DEV).bfloat16()
        out = {name: (off, num) for name, off, num in fb.fise_unet_tensors(u, 2)}
        for name, (off, num) in where.items():
            if name.endswith((".a2.k.w", ".a2.v.w")):
                weights[off:off + num] = (torch.randn(num, generator=g, device=DEV) * 0.05).bfloat16()
        kv = torch.full((int(fb.fise_unet_ctxkv_bytes(u)),), 0x5A, dtype=torch.uint8, device=DEV)
        fb.fise_unet_context_kv(u, weights, ctx, kv)
        x, seen = ctx.float(), 0
        for name, (off, num) in out.items():
            tokens = name.endswith(".ctx_vt")
            w_off, w_num = where[name.replace(".ctx_vt", ".a2.v.w").replace(".ctx_k", ".a2.k.w")]
            w = weights[w_off:w_off + w_num].reshape(-1, ctx_dim).float()
            got = kv[off:off + num].view(torch.bfloat16)
            want, size = x @ w.t(), x.abs() @ w.abs().t()
            if tokens:
                full = got.reshape(B, w.shape[0], -1)
                assert bool((full[:, :, n_ctx:].contiguous().view(torch.int16) == 0x5A5A).all()), "columns past the last token are not touched"
                got = full[:, :, :n_ctx].transpose(1, 2)
            else:
                got = got[: B * n_ctx * w.shape[0]].reshape(B, n_ctx, -1)
            # one rounding to bf16 (2^-9 of the value, twice as much here) and fp32 sums of ctx_dim terms in another order
            assert bool(((got.float() - want).abs() <= want.abs() * 2.0 ** -8 + size * 2.0 ** -18).all()), name
            seen += 1
        assert seen >= 20
    finally:
        fb.fise_unet_destroy(u)
