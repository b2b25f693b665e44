"""Linears of many rows into float rows (64 or 128 rows x 80 columns): whole transformer blocks against the oracle where the last row tile is
partial, full or one batch element's end, on both tile heights and both sides of the rule."""
import pytest
import torch

import test_gpu_blocks as blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


BLOCKS = [
    # name, H, W, C, tile, frac (the rows follow from the mask that it draws)
    ("rows-2106-320", 48, 48, 320, 3, 0.4),              # 64 rows, the last tile of 58
    ("rows-2048-640", 32, 32, 640, 8, 1.0),              # 64 rows, one tile for each CU
    ("rows-4194-320", 66, 72, 320, 3, 0.4),              # 128 rows, the last tile of 98
    ("rows-2432-640", 40, 40, 640, 4, 0.6),              # 128 rows
    ("rows-1926-320", 48, 48, 320, 3, 0.35),             # below the line
]


@pytest.mark.parametrize("case", BLOCKS, ids=[c[0] for c in BLOCKS])
def test_transformer_block(fb, case):
    blocks.test_transformer_block(fb, case)
