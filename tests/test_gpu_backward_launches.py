"""GPU parity of the gradients where several kinds of work share a launch: the pass with the tap gradients in front of the
query side (more than 768 workgroups) and behind it (up to 768), for each layout of the attention; Q, K, V and dO from one
launch with each tile of the product; both depth-wise passes together; dX and the weight gradients in one launch (up to 256
tiles of 128 x 128) and in two; attention by regions and by whole images."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (15, 49, 49, 64, 2, 7, 1),       # 736 workgroups of 64 tokens
    (16, 49, 49, 64, 1, 7, 1),       # 784
    (20, 35, 35, 64, 2, 7, 2),       # 248 workgroups of four regions each
    (63, 35, 35, 64, 2, 7, 2),       # 776
    (2, 20, 30, 64, 2, 2, 1),        # 150 tokens per region, an odd number of column pairs
    (200, 7, 7, 448, 14, 7, 5),      # 128 x 128 tiles
    (90, 7, 7, 320, 10, 7, 3),       # 64 x 128
    (3, 14, 14, 192, 6, 7, 4),       # 64 x 64
    (1, 5, 5, 64, 1, 5, 2),          # one tile, one chunk
    (84, 14, 14, 192, 6, 7, 1),      # dX: 258 tiles of 128 x 128
    (83, 14, 14, 192, 6, 7, 1),      # 256, as tiles of 64 x 64
    (27, 14, 14, 704, 22, 7, 1),     # 252, as tiles of 64 x 128
    (1, 7, 7, 192, 3, 7, 3),
    (79, 7, 7, 64, 2, 7, 5),         # 158 (image, head) pairs: region by region
    (80, 7, 7, 64, 2, 7, 5),         # 160: by whole images
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_shared_launches(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9600 + H * W + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
