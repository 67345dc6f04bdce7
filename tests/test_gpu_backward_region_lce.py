"""GPU parity of the gradients where a workgroup of the attention has its region whole and all routed keys in one block: the depth-wise
parts from the region's halo (57 to 64 tokens, 33 to 64 with more than 1024 regions; k n <= 64), for regions that whole items of 4 x 4 tokens fill, that they do
not, wide and high ones, the most items, halos that the buffers do not hold (the passes of their own), one region on all borders of the map; and the query
side with scores and dP in registers where a wavefront has the region (k n up to 32, and one more)."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (2, 56, 56, 64, 2, 7, 1),        # 8 x 8 tokens
    (1, 49, 63, 128, 4, 7, 1),       # 7 x 9: six items
    (2, 27, 21, 64, 1, 3, 1),        # 9 x 7, a head of 64 channels
    (3, 10, 24, 128, 2, 2, 1),       # 5 x 12
    (1, 12, 12, 192, 6, 2, 1),       # 6 x 6, few regions: the passes
    (2, 24, 88, 64, 2, 8, 1),        # 3 x 11, the same
    (5, 8, 128, 64, 2, 4, 1),        # 2 x 32: more than the buffers hold
    (5, 128, 8, 64, 2, 4, 1),        # 32 x 2
    (1, 36, 4, 64, 2, 4, 1),         # 9 x 1: few tokens
    (1, 33, 2, 64, 2, 1, 1),         # 33 x 2 tokens, one region: too many for one tile
    (2, 33, 1, 64, 2, 1, 1),         # 33 x 1: nine items
    (2, 8, 7, 64, 2, 1, 1),          # 56 tokens, one region
    (2, 9, 7, 64, 2, 1, 1),          # 63, the whole map
    (2, 3, 21, 64, 2, 1, 1),         # six items side by side
    (2, 21, 3, 64, 2, 1, 1),         # above each other
    (17, 16, 224, 64, 2, 8, 1),      # 2 x 28, many regions: seven items, as much as the buffers hold
    (21, 42, 42, 64, 2, 7, 1),       # 6 x 6, many regions
    (17, 24, 88, 64, 2, 8, 1),       # 3 x 11
    (1, 8, 16, 64, 2, 4, 4),         # 8 tokens, 32 keys
    (1, 8, 16, 64, 2, 4, 5),         # 40 keys
    (3, 16, 24, 128, 4, 4, 1),       # 24 tokens
    (2, 16, 32, 128, 2, 4, 1),       # 32
    (2, 7, 7, 64, 2, 7, 32),         # one token, 32 keys
    (2, 7, 7, 64, 1, 7, 33),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_region_convolution(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9900 + H * W + C + k, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
