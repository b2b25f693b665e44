"""Where the key range of the attention is split over workgroups: the scratch size tells, on the host."""
import pytest

from paper_2305_17423_amd import binding as fb


@pytest.mark.parametrize("B,M,n_keys,C,splits", [
    (2, 32, 320, 1280, 1),           # five blocks: one chain, whatever the head
    (1, 1, 320, 1280, 1),
    (2, 32, 321, 1280, 3),           # six and seven blocks of wide heads with few queries
    (2, 32, 448, 1280, 3),
    (2, 262, 384, 1280, 3),          # both sides of the line at head dim 160 (672000 elements), 128 and 80
    (2, 263, 384, 1280, 1),
    (2, 218, 448, 1024, 3),
    (2, 219, 448, 1024, 1),
    (2, 87, 448, 640, 3),
    (2, 88, 448, 640, 1),
    (1, 1, 448, 512, 1),             # heads of 64 and less gain nothing there
    (1, 1, 448, 320, 1),
    (2, 32, 512, 320, 4),            # eight blocks and more, any head
    (2, 4096, 512, 320, 2),
])
def test_key_splits(B, M, n_keys, C, splits):
    def up(n):
        return (n + 255) // 256 * 256
    need = up(splits * B * M * C * 4) + up(splits * B * 8 * M * 8) if splits > 1 else 0
    assert fb.fise_attention_active_workspace_bytes(B, M, n_keys, C, 8) == need
