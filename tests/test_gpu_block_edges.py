"""GPU parity of the block's position kernel at the edges of its tiling: single rows and columns, strips of 2 to 16 rows with
ragged ends, every number of lanes per token, idle lanes (C = 192, 384); of the MLP half in workgroups of 8 wavefronts."""
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


EIGHT = [  # (B, H, W, C, heads, S, k, expansion): MLP half in workgroups of 8 wavefronts, the last one ragged
    (21, 28, 28, 128, 4, 7, 4, 3),
    (19, 29, 31, 128, 4, 1, 1, 1),
    (21, 28, 28, 192, 6, 7, 4, 3),
    (19, 29, 31, 192, 6, 1, 1, 2),
    (84, 14, 14, 256, 8, 7, 4, 3),
    (19, 29, 31, 256, 8, 1, 1, 1),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k,expansion", EIGHT)
def test_mlp_eight_waves(B, H, W, C, heads, S, k, expansion):
    X, P = inputs(B, H, W, C, seed=9650 + H * W + C, expansion=expansion)
    compare_block(X, P, S, k, heads, images=[0, B - 1])
