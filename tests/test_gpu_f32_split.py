"""GPU parity of the float32 family where few rows make the wavefronts of a workgroup share the contraction of its products: rows that no tile
divides, fewer steps than wavefronts and a remainder of them, regions of 1 to 32 tokens with means out of 16 and of 32 rows, bias, GELU and
residual, and both sides of the lines."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_block import compare_block, inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 7, 7, 512, 16, 7, 5),        # 49 rows, one token per region
    (1, 3, 5, 64, 2, 1, 1),          # 15 rows, one region, four steps for eight wavefronts
    (2, 6, 9, 96, 3, 3, 2),          # regions of 6: two to a tile of 16 rows
    (1, 14, 14, 144, 3, 7, 9),       # C = 144: not whole tiles of columns: the other kernel
    (1, 14, 14, 160, 5, 7, 9),       # ten steps
    (2, 16, 16, 256, 8, 4, 3),       # 16 tokens: a tile
    (1, 21, 12, 192, 6, 3, 2),       # 28: 32 rows
    (1, 8, 16, 256, 8, 2, 2),        # 32
    (1, 32, 16, 128, 4, 4, 2),       # 32, 48 tiles of 64 x 64 at K = 128: the other kernel
    (1, 34, 4, 96, 3, 2, 1),         # 34: the other kernel
    (3, 14, 14, 256, 8, 7, 6),       # 32 rows, 588 of them
    (3, 14, 28, 256, 8, 7, 6),       # beyond
    (2, 8, 8, 768, 24, 8, 2),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_forward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9980 + H * W + C, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, heads, "generic")


@pytest.mark.parametrize("B,H,W,C,heads,S,k,e", [
    (1, 7, 7, 512, 16, 7, 5, 3),
    (1, 3, 5, 64, 2, 1, 1, 1),
    (2, 14, 14, 128, 4, 7, 6, 2),
    (1, 28, 28, 96, 3, 7, 4, 4),
])
def test_block(B, H, W, C, heads, S, k, e):
    X, P = inputs(B, H, W, C, seed=9981 + H * W + C, expansion=e, dtype="f32")
    compare_block(X, P, S, k, heads, dtype="f32")


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (1, 7, 7, 768, 12, 7, 44),
    (1, 3, 5, 64, 2, 1, 1),
    (2, 6, 9, 96, 3, 3, 2),
    (2, 14, 14, 256, 8, 7, 4),
    (2, 14, 14, 512, 16, 7, 4),
    (1, 28, 28, 128, 4, 7, 4),
])
def test_backward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9982 + H * W + C, dtype="f32")
    compare_backward(X, Wqkv, Wo, Wlce, "f32", heads, S, k, path="generic")
