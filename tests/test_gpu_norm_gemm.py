"""Products behind a normalisation as one launch (widths 320, 640 and 1280): whole blocks and layers against the oracle where the rows or
columns of a workgroup's tile run out: a handful of rows, tiles whose pixels are no runs of four, batch elements that end
inside a row tile, and as many rows as make several column tiles a workgroup."""
import pytest
import torch

import test_gpu_attention as attention
import test_gpu_blocks as blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


BLOCKS = [
    # name, H, W, C, tile, frac
    ("a-few-pixels-320", 8, 8, 320, 1, 0.05),
    ("tile3-320", 12, 18, 320, 3, 0.3),
    ("tile2-320", 16, 24, 320, 2, 0.2),
    ("rows-past-2048-320", 64, 64, 320, 8, 0.5),
    ("tile5-640", 20, 20, 640, 5, 0.1),
    ("a-few-pixels-640", 8, 16, 640, 1, 0.05),
    ("most-of-a-map-640", 32, 32, 640, 4, 0.8),
    ("tile3-1280", 12, 6, 1280, 3, 0.2),
    ("a-few-pixels-1280", 8, 8, 1280, 1, 0.05),
    ("most-of-a-map-1280", 16, 16, 1280, 2, 0.8),
]


@pytest.mark.parametrize("case", BLOCKS, ids=[c[0] for c in BLOCKS])
def test_transformer_block(fb, case):
    blocks.test_transformer_block(fb, case)


@pytest.mark.parametrize("C,heads,H,W,t,frac,cross", [(1280, 8, 8, 8, 1, 0.1, False), (640, 8, 12, 12, 3, 0.3, False), (320, 8, 24, 16, 1, 0.05, True),
                                                       (1280, 8, 16, 16, 4, 0.8, False), (640, 8, 16, 8, 2, 0.3, True), (320, 8, 48, 56, 4, 0.6, False)])
def test_attention_layer(fb, C, heads, H, W, t, frac, cross):
    attention.test_masked_attention_layer(fb, C, heads, H, W, t, frac, cross)
