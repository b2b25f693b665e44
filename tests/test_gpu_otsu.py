"""GPU parity of the Otsu threshold at the sizes where its chunks and bins can go wrong: counts and sums of every bin bit for bit
in index order, threshold and mask against the oracle."""
import numpy as np
import pytest
import torch

from oracle import fise_oracle as fo
from helpers import DEV, dev

pytestmark = pytest.mark.gpu
BINS = 257


@pytest.mark.parametrize("n", [1, 2, 63, 1023, 1024, 1025, 4096, 9216, 255, 4095, 4097, 8191, 12289])
@pytest.mark.parametrize("shape", ["uniform", "one-bin-and-one", "two-clusters"])
def test_otsu_bins_in_index_order(n, shape):
    from paper_2305_17423_amd import binding as fb
    rng = np.random.default_rng(n)
    if shape == "uniform":
        d = rng.random(n)
    elif shape == "one-bin-and-one":                    # all but one value in the lowest bin: one chain of n additions
        d = rng.random(n) * 1e-3
        d[n // 2] = 1.0
    else:
        d = np.where(rng.random(n) < 0.3, 0.8, 0.1) + 0.05 * rng.random(n)
    d = d.astype(np.float32)
    eps, pix = torch.full((1,), -1.0, device=DEV), torch.full((n,), 7, dtype=torch.uint8, device=DEV)
    ws = torch.full((fb.fise_otsu_workspace_bytes(),), 0xA5, dtype=torch.uint8, device=DEV)
    fb.fise_otsu_mask(dev(d), eps, pix, ws)
    v = fo.normalize_minmax(d.astype(np.float64))
    cnt, tot = np.zeros(BINS), np.zeros(BINS)
    for x in v:
        k = int(np.floor(x * 256.0))
        cnt[k] += 1.0
        tot[k] += x
    got = ws.cpu().numpy()[:8 * (2 + 2 * BINS)].view(np.float64)
    assert np.array_equal(got[2:2 + BINS], cnt) and np.array_equal(got[2 + BINS:], tot)
    want, mask = fo.otsu_threshold(v)
    assert float(eps.item()) == np.float32(want)
    assert np.array_equal(pix.cpu().numpy(), mask.reshape(-1).astype(np.uint8))


def _trailing_zeros(x):
    m = int(np.float64(x).view(np.int64)) & (1 << 52) - 1
    return 52 if m == 0 else (m & -m).bit_length() - 1


@pytest.mark.parametrize("n", [33, 257, 4096, 9216])
@pytest.mark.parametrize("shape", ["zeros", "half-places", "tiny-then-large", "steps"])
def test_otsu_sums_where_additions_round_otherwise(n, shape):
    """Sums that start at zero, additions half way between two places of the sum (one value over and over whose last set bit is the
    ninth or higher: 2^8 of them in a row tie), values far below the sum, few distinct values: every bin bit for bit."""
    from paper_2305_17423_amd import binding as fb
    rng = np.random.default_rng(n)
    d = (rng.random(n) * 3e-3).astype(np.float32)
    if shape == "zeros":
        d[rng.random(n) < 0.9] = 0.0
    elif shape == "half-places":
        while not 8 <= _trailing_zeros(np.float64(np.float32(c := rng.random() * 3e-3)) / np.float64(np.float32(0.9))) <= 11:
            pass
        d[:] = c
    elif shape == "tiny-then-large":
        d[: n // 2] *= 1e-30
    else:
        d = (np.round(d * 4000) / 3700).astype(np.float32) * np.float32(0.99)
    d[0], d[n - 1] = 0.0, 0.9
    eps, pix = torch.full((1,), -1.0, device=DEV), torch.full((n,), 7, dtype=torch.uint8, device=DEV)
    ws = torch.full((fb.fise_otsu_workspace_bytes(),), 0xA5, dtype=torch.uint8, device=DEV)
    fb.fise_otsu_mask(dev(d), eps, pix, ws)
    v = fo.normalize_minmax(d.astype(np.float64))
    tot = np.zeros(BINS)
    for x in v:
        tot[int(np.floor(x * 256.0))] += x
    got = ws.cpu().numpy()[:8 * (2 + 2 * BINS)].view(np.float64)
    assert np.array_equal(got[2 + BINS:], tot)


def test_otsu_sums_that_cross_a_power_of_two_behind_a_tie():
    """The lowest bin's sum a few places below 2, then ties and whole places that take it across within one block (minimum 0 and maximum 1: a value is what is
    added).  A few in a thousand of these sums differ where a scan that has passed the power of two is used any further."""
    from paper_2305_17423_amd import binding as fb
    rng = np.random.default_rng(1)
    eps, pix = torch.zeros(1, device=DEV), torch.zeros(2048, dtype=torch.uint8, device=DEV)
    got, want = [], []
    for _ in range(1500):
        rest = 2 ** 43 - int(rng.integers(1, 65))                # of 2^-9, in places of 2^-52: 2 - k 2^-52 in all
        head = [2.0 ** -9] * 1023 + [2.0 ** (b - 52) for b in range(42, -1, -1) if rest >> b & 1]
        v = np.zeros(-(-len(head) // 256) * 256 + 257)
        v[:len(head)] = head
        v[-257:-1] = np.where(rng.random(256) < 0.125, 0, rng.integers(1, 7, 256)) * np.where(rng.random(256) < 0.66, 2.0 ** -53, 2.0 ** -52)
        v[-1] = 1.0
        ws = torch.zeros(fb.fise_otsu_workspace_bytes(), dtype=torch.uint8, device=DEV)
        fb.fise_otsu_mask(dev(v.astype(np.float32)), eps, pix, ws)
        got.append(ws[8 * (2 + BINS):8 * (3 + BINS)])
        want.append(np.cumsum(v[:-1])[-1])                       # one addition after the other
    got = torch.stack(got).cpu().numpy().view(np.float64)[:, 0]
    assert np.array_equal(got, np.array(want)), int((got != np.array(want)).sum())


@pytest.mark.parametrize("n", [1, 70, 5000])
@pytest.mark.parametrize("shape", ["equal", "nan", "negative-nan", "all-nan", "inf", "minus-inf", "both-inf"])
def test_otsu_values_without_a_range(n, shape):
    """Equal values are all zero and above the threshold of zero.  NaN are left out of minimum and maximum and, like all values of an infinite range but
    its infinities, belong to the lowest bin; a sum they are part of is NaN, whose threshold is zero, and they are not above it."""
    from paper_2305_17423_amd import binding as fb
    d = np.full(n, 0.25, np.float32) if shape == "equal" else np.random.default_rng(n).random(n).astype(np.float32)
    if shape == "all-nan":
        d[:] = np.nan
    elif "nan" in shape:
        d[n // 2] = np.array([0xffc00000], np.uint32).view(np.float32)[0] if shape == "negative-nan" else np.nan
    if shape in ("inf", "both-inf"):
        d[n // 2] = np.inf
    if shape in ("minus-inf", "both-inf"):
        d[n // 3] = -np.inf
    eps, pix = torch.full((1,), -1.0, device=DEV), torch.full((n,), 7, dtype=torch.uint8, device=DEV)
    ws = torch.full((fb.fise_otsu_workspace_bytes(),), 0xA5, dtype=torch.uint8, device=DEV)
    fb.fise_otsu_mask(dev(d), eps, pix, ws)
    with np.errstate(invalid="ignore", over="ignore"):
        x = d.astype(np.float64)
        lo, hi = np.fmin.reduce(x, initial=1e300), np.fmax.reduce(x, initial=-1e300)
        v = (x - lo) / (hi - lo) if hi > lo else np.zeros(n)
    k = np.where(np.isnan(v), 0, np.floor(np.where(np.isnan(v), 0, v) * 256)).astype(int)
    got = ws.cpu().numpy()[:8 * (2 + 2 * BINS)].view(np.float64)
    assert np.array_equal(got[2:2 + BINS], np.bincount(k, minlength=BINS))
    tot = np.zeros(BINS)
    for i, b in enumerate(k):
        tot[b] += v[i]
    assert np.array_equal(got[2 + BINS:], tot, equal_nan=True)
    if shape == "equal" or np.isnan(tot).any():
        assert float(eps.item()) == 0.0
    assert np.array_equal(pix.cpu().numpy(), (v >= float(eps.item())).astype(np.uint8))
