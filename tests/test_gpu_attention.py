"""GPU parity: active-query attention, the masked attention sub-layer and the context K/V projection."""
import math

import numpy as np
import pytest
import torch

from oracle import fise_oracle as fo
from paper_2305_17423_amd import workloads as wl
from helpers import DEV, TOL, dev, host, rel_err, idx_dev, active_mask, check_map

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def vt_dev(V, n_stride=None, poison=False):
    """[B, N, C] -> device transposed [B, C, n_stride]; padding columns hold garbage on request."""
    B, N, C = V.shape
    ns = N if n_stride is None else n_stride
    buf = np.zeros((B, C, ns), np.float32)
    if poison:
        buf[:] = np.nan
    buf[:, :, :N] = V.transpose(0, 2, 1)
    return dev(buf, "bf16")


# B, queries, keys, channels, heads, form without scratch, form with it: 0 the kernel for few queries, else the key splits of the one for many
# (test_attention_splits.py asks the launcher for both)
ACTIVE = [
    (2, 200, 4096, 320, 8, 0, 8),     # config 3 shape: d = 40, ragged query count
    (2, 64, 1024, 640, 8, 0, 8),      # d = 80
    (1, 37, 256, 1280, 8, 0, 0),      # d = 160
    (2, 33, 77, 320, 8, 0, 0),        # cross-attention: 77 keys (tail block), stride 80
    (2, 16, 64, 32, 4, 1, 1),         # d = 8
    (1, 130, 200, 128, 4, 0, 0),      # d = 32, keys not a multiple of 64
    (1, 1, 8, 64, 4, 0, 0),           # one query, one partial block
    (2, 16, 448, 1280, 8, 0, 0),      # seven blocks of wide heads, few queries: scratch for three key splits, not used
    (1, 40, 330, 1024, 8, 0, 0),      # d = 128, six blocks, the last partial
    # few queries (one launch, the keys dealt out among the waves of a workgroup): key counts around 32 and around one and two turns of the
    # waves, query counts around the tile of 32, every head dim that has a padding of its own
    (1, 1, 1, 64, 8, 0, 0),           # one query, one key, d = 8
    (2, 31, 31, 96, 4, 0, 0),         # d = 24
    (1, 32, 32, 320, 8, 0, 0),        # d = 40
    (2, 33, 33, 384, 8, 0, 0),        # d = 48
    (2, 64, 95, 256, 4, 0, 0),        # d = 64
    (2, 64, 63, 256, 4, 1, 1),
    (1, 65, 65, 640, 8, 0, 0),        # d = 80
    (2, 5, 129, 768, 8, 0, 0),        # d = 96, five waves with keys
    (1, 40, 255, 416, 4, 0, 0),       # d = 104
    (2, 48, 256, 1024, 8, 0, 0),      # d = 128, one turn of the waves
    (1, 17, 257, 1088, 8, 0, 0),      # d = 136, a second turn of one key
    (2, 100, 289, 1280, 8, 0, 0),     # d = 160
    (2, 300, 520, 320, 8, 0, 0),      # more workgroups than CUs, three turns
    (4, 12, 77, 1280, 8, 0, 0),
    # many queries: launches that use fewer key splits than their scratch is laid out for, or none, around the lines where the count changes and
    # with last splits of one partial key block
    (2, 700, 800, 640, 8, 1, 1),      # six splits fit, one is used
    (2, 576, 576, 1280, 8, 1, 1),     # four, one
    (2, 600, 120, 256, 8, 1, 1),      # d = 32
    (2, 520, 120, 768, 8, 1, 1),      # d = 96
    (1, 130, 2000, 256, 4, 0, 16),    # sixteen, all
    (1, 700, 1500, 416, 4, 0, 6),     # twelve, six
    (2, 384, 4033, 320, 8, 0, 5),     # fourteen, five, the last block one key
    (2, 688, 1281, 640, 8, 0, 2),     # seven, between
    (1, 3, 577, 1280, 8, 0, 5),       # d = 160, ten blocks in fives of two, the last partial
    (2, 130, 1000, 1024, 8, 0, 8),    # d = 128, a second query tile of two
]


@pytest.mark.parametrize("B,M,N,C,heads", [c[:5] for c in ACTIVE])
def test_attention_active(fb, B, M, N, C, heads):
    rng = np.random.default_rng(4000 + M + N)
    q = wl.normal(rng, (B, M, C), 1.0, "bf16"); K = wl.normal(rng, (B, N, C), 1.0, "bf16"); V = wl.normal(rng, (B, N, C), 1.0, "bf16")
    want = fo.attention_active(q, K, V, heads)
    ns = (N + 7) // 8 * 8
    out = torch.zeros((B, M, C), dtype=torch.bfloat16, device=DEV)
    fb.fise_attention_active(dev(q, "bf16"), dev(K, "bf16"), vt_dev(V, ns, poison=True), heads, 1 / math.sqrt(C // heads), out, n_keys=N)
    err = rel_err(host(out), want)
    assert err <= TOL["bf16"], err
    # with scratch the key range may be split over workgroups and merged: same result
    nb = fb.fise_attention_active_workspace_bytes(B, M, N, C, heads)
    ws = torch.full((max(nb, 256),), 0x7F, dtype=torch.uint8, device=DEV)
    out2 = torch.zeros((B, M, C), dtype=torch.bfloat16, device=DEV)
    fb.fise_attention_active(dev(q, "bf16"), dev(K, "bf16"), vt_dev(V, ns, poison=True), heads, 1 / math.sqrt(C // heads), out2, n_keys=N, workspace=ws)
    err2 = rel_err(host(out2), want)
    assert err2 <= TOL["bf16"], err2


# The partial block is the first one (up to 63 keys) or a later one.  35 queries of two heads run on either kernel, by d and N; 520 of eight on that for
# many queries at every d and N (test_attention_splits.py says so).
PARTIAL_D, PARTIAL_N, PARTIAL_QUERIES = [40, 72, 80, 128, 136, 160], [1, 9, 31, 33, 56, 57, 63, 64, 65, 120], [(35, 2), (520, 8)]


@pytest.mark.parametrize("M,heads", PARTIAL_QUERIES)
@pytest.mark.parametrize("d", PARTIAL_D)
@pytest.mark.parametrize("N", PARTIAL_N)
def test_attention_partial_key_blocks(fb, d, N, M, heads):
    """Head dims of the constant instantiations (80, 160), of the same tiles with the head dim as an argument (72, 136) and of padded tiles; key padding
    of V^T holds NaN."""
    rng = np.random.default_rng(4050 + 200 * d + N)
    B = 2
    C = d * heads
    q = wl.normal(rng, (B, M, C), 1.0, "bf16"); K = wl.normal(rng, (B, N, C), 1.0, "bf16"); V = wl.normal(rng, (B, N, C), 1.0, "bf16")
    want = fo.attention_active(q, K, V, heads)
    out = torch.zeros((B, M, C), dtype=torch.bfloat16, device=DEV)
    fb.fise_attention_active(dev(q, "bf16"), dev(K, "bf16"), vt_dev(V, (N + 7) // 8 * 8, poison=True), heads, 1 / math.sqrt(d), out, n_keys=N)
    assert rel_err(host(out), want) <= TOL["bf16"]


# Long key ranges of heads of 40, 80 and 160 (attention_turns_kernel; test_attention_splits.py says so), in one part and in several: whole turns, a last turn of
# one key, of one more than a 32-key block and of all but one; queries on both sides of a tile of 128.
TURNS = [(40, 512, 513), (40, 513, 1500), (40, 545, 1500), (40, 2199, 600), (40, 4160, 257), (80, 512, 640), (80, 513, 513), (80, 545, 600), (80, 1087, 700),
         (160, 512, 513), (160, 513, 640), (160, 545, 600), (160, 1087, 700), (160, 2199, 513),
         # heads of 40 and 80 from twelve key blocks a part on: the same ends
         (40, 768, 1500), (40, 769, 1500), (40, 801, 1500), (40, 895, 1500), (40, 4161, 700), (80, 768, 1500), (80, 769, 1500), (80, 801, 1500), (80, 895, 1500), (80, 4127, 700)]


@pytest.mark.parametrize("d,N,M", TURNS)
def test_attention_long_key_ranges(fb, d, N, M):
    rng = np.random.default_rng(4070 + d + N)
    B, heads = 2, 8
    C = d * heads
    q = wl.normal(rng, (B, M, C), 1.0, "bf16"); K = wl.normal(rng, (B, N, C), 1.0, "bf16"); V = wl.normal(rng, (B, N, C), 1.0, "bf16")
    want = fo.attention_active(q, K, V, heads)
    Vd = vt_dev(V, (N + 7) // 8 * 8 + 8, poison=True)
    for scratch in (False, True):
        ws = torch.full((max(fb.fise_attention_active_workspace_bytes(B, M, N, C, heads), 256),), 0x7F, dtype=torch.uint8, device=DEV) if scratch else None
        out = torch.zeros((B, M, C), dtype=torch.bfloat16, device=DEV)
        fb.fise_attention_active(dev(q, "bf16"), dev(K, "bf16"), Vd, heads, 1 / math.sqrt(d), out, n_keys=N, workspace=ws)
        assert rel_err(host(out), want) <= TOL["bf16"], scratch


# The same columns as ACTIVE: splits on both sides of the numbers of parts that a merge requests at once, the most there are among them.
MERGES = [(1, 30, 1100, 160, 1, 0, 9), (2, 70, 1500, 40, 1, 0, 12), (1, 36, 2226, 80, 2, 0, 12), (1, 20, 3000, 128, 2, 0, 16), (1, 20, 5000, 80, 2, 0, 27), (1, 20, 4096, 80, 2, 0, 32)]


@pytest.mark.parametrize("B,M,N,C,heads", [c[:5] for c in MERGES])
def test_attention_merges(fb, B, M, N, C, heads):
    test_attention_active(fb, B, M, N, C, heads)


def test_attention_closed_forms_on_device(fb):
    rng = np.random.default_rng(4100)
    B, M, N, C, heads = 1, 40, 300, 320, 8
    q = wl.normal(rng, (B, M, C), 1.0, "bf16"); K = wl.normal(rng, (B, N, C), 1.0, "bf16")
    vrow = wl.normal(rng, (1, 1, C), 1.0, "bf16")
    V = np.broadcast_to(vrow, (B, N, C)).copy()
    out = torch.zeros((B, M, C), dtype=torch.bfloat16, device=DEV)
    fb.fise_attention_active(dev(q, "bf16"), dev(K, "bf16"), vt_dev(V, 304), heads, 1 / math.sqrt(40), out, n_keys=N)
    assert rel_err(host(out), np.broadcast_to(vrow, (B, M, C))) < 1e-2          # constant V -> that constant
    # sharply peaked logits: output = V of the matching key
    Kp = np.zeros((1, 64, 64), np.float32); qp = np.zeros((1, 64, 64), np.float32)
    for i in range(64):
        Kp[0, i, i] = 16.0; qp[0, i, i] = 16.0
    Vp = wl.normal(rng, (1, 64, 64), 1.0, "bf16")
    out = torch.zeros((1, 64, 64), dtype=torch.bfloat16, device=DEV)
    fb.fise_attention_active(dev(qp, "bf16"), dev(Kp, "bf16"), vt_dev(Vp), 1, 1 / 8.0, out)
    assert rel_err(host(out), Vp) < 1e-2


@pytest.mark.parametrize("C,heads,H,W,t,frac,cross", [(320, 8, 64, 64, 4, 0.05, False), (320, 8, 64, 64, 4, 0.2, False),
                                                       (320, 8, 64, 64, 4, 0.1, True), (640, 8, 32, 32, 4, 0.1, False),
                                                       (64, 4, 8, 8, 2, 0.3, False),
                                                       # queries, keys and values behind the LayerNorm in one launch, see test_gpu_blocks.TR_CASES
                                                       (1280, 8, 8, 8, 1, 0.1, False), (640, 8, 12, 12, 3, 0.3, False), (320, 8, 24, 16, 1, 0.05, True),
                                                       (1280, 8, 16, 16, 4, 0.8, False), (640, 8, 16, 8, 2, 0.3, True), (320, 8, 48, 56, 4, 0.6, False)])
def test_masked_attention_layer(fb, C, heads, H, W, t, frac, cross):
    rng = np.random.default_rng(4200 + C + int(frac * 100) + cross)
    B, dt, Dc, n_ctx = 2, "bf16", 768, 77
    x_old = wl.normal(rng, (B, H, W, C), 1.0, dt)
    pixm = wl.ellipse_pixels(rng, H, W, frac)
    x_new = wl.perturb(rng, x_old, pixm, 1.0, dt)
    _, idx = fo.tiles_from_pixels(pixm, t)
    g = wl.normal(rng, (C,), 0.02, dt, mean=1.0); b0 = wl.normal(rng, (C,), 0.02, dt)
    s = 1 / math.sqrt(C)
    wq, wo = wl.normal(rng, (C, C), s, dt), wl.normal(rng, (C, C), s, dt)
    bo = wl.normal(rng, (C,), 0.02, dt)
    full = fo.full_index(H, W, t)
    if cross:
        ctx = wl.normal(rng, (B, n_ctx, Dc), 1.0, dt)
        wk, wv = wl.normal(rng, (C, Dc), 1 / math.sqrt(Dc), dt), wl.normal(rng, (C, Dc), 1 / math.sqrt(Dc), dt)
        Kc, Vc = fo.context_kv(ctx, wk, wv, dt)
        Kd = torch.zeros((B, n_ctx, C), dtype=torch.bfloat16, device=DEV); Vd = torch.zeros((B, C, 80), dtype=torch.bfloat16, device=DEV)
        fb.fise_context_kv(dev(ctx, dt), dev(wk, dt), dev(wv, dt), Kd, Vd)
        assert rel_err(host(Kd), Kc) <= TOL[dt] and rel_err(host(Vd)[:, :, :n_ctx].transpose(0, 2, 1), Vc) <= TOL[dt]
        y_cache = wl.normal(rng, (B, H, W, C), 1.0, dt)
        want = y_cache.astype(np.float64).copy()
        fo.masked_attention_block(x_new, g, b0, wq, None, None, wo, bo, heads, None, None, Kc, Vc, idx, t, want, dt)
        y = dev(y_cache, dt)
        ws = torch.zeros(fb.fise_masked_attention_workspace_bytes(B, C, idx.size, t), dtype=torch.uint8, device=DEV)
        fb.fise_masked_attention(dev(x_new, dt), dev(g, dt), dev(b0, dt), dev(wq, dt), None, None, dev(wo, dt), dev(bo, dt), heads,
                                 None, None, dev(Kc, dt), vt_dev(Vc, 80), n_ctx, idx_dev(idx), idx.size, t, y, ws)
        check_map(host(y), want, y_cache.astype(np.float64), active_mask(idx, t, H, W), TOL[dt], "cross")
        return
    wk, wv = wl.normal(rng, (C, C), s, dt), wl.normal(rng, (C, C), s, dt)
    # caches of the old generation, from the oracle's dense pass
    K0 = np.zeros((B, H * W, C)); V0 = np.zeros((B, H * W, C)); y0 = np.zeros((B, H, W, C))
    fo.masked_attention_block(x_old, g, b0, wq, wk, wv, wo, bo, heads, K0, V0, None, None, full, t, y0, dt)
    Kw, Vw, want = K0.copy(), V0.copy(), y0.copy()
    fo.masked_attention_block(x_new, g, b0, wq, wk, wv, wo, bo, heads, Kw, Vw, None, None, idx, t, want, dt)
    Kd, Vd, y = dev(K0, dt), vt_dev(V0), dev(y0, dt)
    ws = torch.zeros(fb.fise_masked_attention_workspace_bytes(B, C, idx.size, t), dtype=torch.uint8, device=DEV)
    args = (dev(x_new, dt), dev(g, dt), dev(b0, dt), dev(wq, dt), dev(wk, dt), dev(wv, dt), dev(wo, dt), dev(bo, dt), heads,
            Kd, Vd, None, None, 0, idx_dev(idx), idx.size, t, y, ws)
    fb.fise_masked_attention(*args)
    act = active_mask(idx, t, H, W)
    got = host(y)
    check_map(got, want, y0, act, TOL[dt], "self")
    av = act.reshape(-1)
    gK, gV = host(Kd), host(Vd).transpose(0, 2, 1)
    assert rel_err(gK[:, av], Kw[:, av]) <= TOL[dt] and np.array_equal(gK[:, ~av], K0[:, ~av])
    assert rel_err(gV[:, av], Vw[:, av]) <= TOL[dt] and np.array_equal(gV[:, ~av], V0[:, ~av])
    fb.fise_masked_attention(*args)                                             # idempotent (K/V refresh included)
    assert np.array_equal(host(y), got) and np.array_equal(host(Kd), gK)


@pytest.mark.parametrize("C,heads,H,W,t,frac", [(320, 8, 64, 64, 4, 0.10), (320, 8, 64, 64, 4, 0.02), (640, 8, 32, 32, 4, 0.25),
                                                 (1280, 8, 8, 8, 1, 0.3), (64, 4, 8, 8, 2, 0.3)])
def test_keys_restricted_attention_layer(fb, C, heads, H, W, t, frac):
    """Active queries x active keys (no K/V cache): element by element against the oracle, cache kept elsewhere,
    idempotent, full mask == the cached form with every key, empty mask touches nothing.  Also prints how far the
    restricted form is from the full-key form on this synthetic input (information, not a check)."""
    rng = np.random.default_rng(4300 + C + int(frac * 100))
    B, dt = 2, "bf16"
    x_old = wl.normal(rng, (B, H, W, C), 1.0, dt)
    pixm = wl.ellipse_pixels(rng, H, W, frac)
    x_new = wl.perturb(rng, x_old, pixm, 1.0, dt)
    _, idx = fo.tiles_from_pixels(pixm, t)
    full = fo.full_index(H, W, t)
    g = wl.normal(rng, (C,), 0.02, dt, mean=1.0); b0 = wl.normal(rng, (C,), 0.02, dt)
    s = 1 / math.sqrt(C)
    wq, wk, wv, wo = (wl.normal(rng, (C, C), s, dt) for _ in range(4))
    bo = wl.normal(rng, (C,), 0.02, dt)
    y_cache = wl.normal(rng, (B, H, W, C), 1.0, dt)
    want = fo.masked_attention_restricted(x_new, g, b0, wq, wk, wv, wo, bo, heads, idx, t, y_cache.astype(np.float64).copy(), dt)
    y = dev(y_cache, dt)
    ws = torch.full((fb.fise_masked_attention_restricted_workspace_bytes(B, C, full.size, t),), 0xFF, dtype=torch.uint8, device=DEV)
    args = (dev(x_new, dt), dev(g, dt), dev(b0, dt), dev(wq, dt), dev(wk, dt), dev(wv, dt), dev(wo, dt), dev(bo, dt), heads)
    fb.fise_masked_attention_restricted(*args, idx_dev(idx), idx.size, t, y, ws)
    act = active_mask(idx, t, H, W)
    got = host(y)
    e = check_map(got, want, y_cache.astype(np.float64), act, TOL[dt], "keys-restricted")
    fb.fise_masked_attention_restricted(*args, idx_dev(idx), idx.size, t, y, ws)
    assert np.array_equal(host(y), got)                                        # idempotent
    y0 = dev(y_cache, dt)
    fb.fise_masked_attention_restricted(*args, idx_dev(idx), 0, t, y0, ws)
    assert np.array_equal(host(y0), y_cache)                                   # empty mask
    # full mask: every key is active, so this is ordinary attention = the cached form driven with the full list
    Kf = np.zeros((B, H * W, C)); Vf = np.zeros((B, H * W, C))
    wantf = fo.masked_attention_block(x_new, g, b0, wq, wk, wv, wo, bo, heads, Kf, Vf, None, None, full, t, np.zeros((B, H, W, C)), dt)
    yf = torch.zeros((B, H, W, C), dtype=torch.bfloat16, device=DEV)
    fb.fise_masked_attention_restricted(*args, idx_dev(full), full.size, t, yf, ws)
    assert rel_err(host(yf), wantf) <= TOL[dt]
    # information: distance between the two readings at the active positions (full keys from the old generation's cache)
    K0 = np.zeros((B, H * W, C)); V0 = np.zeros((B, H * W, C))
    fo.masked_attention_block(x_old, g, b0, wq, wk, wv, wo, bo, heads, K0, V0, None, None, full, t, np.zeros((B, H, W, C)), dt)
    allk = fo.masked_attention_block(x_new, g, b0, wq, wk, wv, wo, bo, heads, K0, V0, None, None, idx, t, y_cache.astype(np.float64).copy(), dt)
    print(f"C={C} {H}x{W} {idx.size} tiles: device vs oracle {e:.2e}; restricted vs all-keys reading (oracle) "
          f"{rel_err(want[:, act], allk[:, act]):.2e}")
