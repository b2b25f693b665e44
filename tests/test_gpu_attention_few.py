"""Attention of few queries (one launch, the keys dealt out among the waves of a workgroup): key counts around 32 and around one and two turns of
the waves, query counts around the tile of 32, every head dim that has a padding of its own."""
import pytest
import torch

import test_gpu_attention as attention

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2305_17423_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


@pytest.mark.parametrize("B,M,N,C,heads", [
    (1, 1, 1, 64, 8),            # one query, one key, d = 8
    (2, 31, 31, 96, 4),          # d = 24
    (1, 32, 32, 320, 8),         # d = 40
    (2, 33, 33, 384, 8),         # d = 48
    (2, 64, 63, 256, 4),         # d = 64
    (1, 65, 65, 640, 8),         # d = 80
    (2, 5, 129, 768, 8),         # d = 96, five waves with keys
    (1, 40, 255, 416, 4),        # d = 104
    (2, 48, 256, 1024, 8),       # d = 128, one turn of the waves
    (1, 17, 257, 1088, 8),       # d = 136, a second turn of one key
    (2, 100, 289, 1280, 8),      # d = 160
    (2, 300, 520, 320, 8),       # more workgroups than CUs, three turns
    (4, 12, 77, 1280, 8),
])
def test_attention_active(fb, B, M, N, C, heads):
    attention.test_attention_active(fb, B, M, N, C, heads)
