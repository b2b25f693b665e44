"""3x3 convolutions on tiles of 64 or 128 rows x 80 columns (which form a case takes is the launcher's choice; at these sizes it is this one): row
tiles whose last strips are absent or belong to the next batch element, one chunk of channels and odd and even numbers of them, source changes,
and the shortcut's side product of whole blocks."""
import pytest
import torch

import test_gpu_blocks as blocks
import test_gpu_wave_gemm as gemm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


CASES = [
    # name, B, H(out), W(out), C0, C1, Cout, k, stride, ups, tile, tiles, temb, res
    ("wide8-128-one-chunk-tail", 1, 96, 80, 64, 0, 320, 3, 1, 0, 8, 119, True, True),
    ("wide8-128-sources-two-batches", 2, 64, 64, 64, 64, 320, 3, 1, 0, 8, 59, True, False),
    ("wide8-128-three-chunks", 2, 64, 64, 64, 128, 320, 3, 1, 0, 8, 64, False, True),
    ("wide8-64", 1, 64, 64, 192, 0, 320, 3, 1, 0, 8, 57, True, True),
    ("wide8-64-narrow-map", 2, 32, 64, 64, 64, 640, 3, 1, 0, 8, 15, False, True),
    ("wide4-64-tail", 1, 48, 40, 64, 128, 640, 3, 1, 0, 4, 113, True, True),
    ("wide4-64-two-batches", 2, 40, 24, 128, 0, 1280, 3, 1, 0, 4, 31, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_conv(fb, case):
    gemm.test_wave_gemm_edges(fb, case)


@pytest.mark.parametrize("case", [
    # name, B, H, W, C0, C1, Cout, tile, frac, weight std
    ("wide8-64-shortcut", 2, 32, 32, 320, 64, 640, 8, 0.9, 0.02),
    ("wide8-128-shortcut", 2, 64, 64, 64, 128, 320, 8, 0.7, 0.03),
    ("wide4-64-shortcut", 2, 32, 32, 128, 192, 640, 4, 0.8, 0.02),
], ids=lambda c: c[0])
def test_resnet_block(fb, case):
    blocks.test_resnet_block(fb, case)
