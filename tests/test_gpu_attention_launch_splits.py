"""Attention of many queries: launches that use fewer key splits than their scratch is laid out for, or none, around the lines where the count
changes and with last splits of one partial key block."""
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
    (2, 700, 800, 640, 8),       # six splits fit, one is used
    (2, 576, 576, 1280, 8),      # four, one
    (1, 130, 2000, 256, 4),      # sixteen, all
    (1, 700, 1500, 416, 4),      # twelve, six
    (2, 384, 4033, 320, 8),      # fourteen, five, the last block one key
    (2, 688, 1281, 640, 8),      # seven, between
])
def test_attention_active(fb, B, M, N, C, heads):
    attention.test_attention_active(fb, B, M, N, C, heads)
