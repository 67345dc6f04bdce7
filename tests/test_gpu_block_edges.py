"""GPU parity of the block's position kernel at the edges of its tiling: single rows and columns, strips of 2 to 16 rows with
ragged ends, every number of lanes per token, idle lanes (C = 192, 384)."""
import pytest

from test_gpu_block import compare_block, inputs

pytestmark = pytest.mark.gpu

EDGES = [  # (B, H, W, C, heads, S, k)
    (2, 1, 9, 64, 1, 1, 1),
    (1, 35, 1, 128, 4, 1, 1),
    (1, 17, 3, 192, 6, 1, 1),
    (48, 34, 20, 64, 2, 2, 1),
    (5, 19, 5, 256, 8, 1, 1),
    (3, 6, 11, 384, 12, 1, 1),
    (2, 5, 7, 512, 16, 1, 1),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", EDGES)
def test_position_strips(B, H, W, C, heads, S, k):
    X, P = inputs(B, H, W, C, seed=9600 + H * W + C, expansion=1)
    compare_block(X, P, S, k, heads, images=[0, B - 1])
