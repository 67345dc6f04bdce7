"""GPU parity of the bf16 products of few rows, whose wavefronts share the contraction: rows that no tile divides, contractions of fewer steps than a
wavefront's ring holds, of several rounds of it and a remainder, regions of 1 to 32 tokens with means, padded maps, bias, GELU and residual, the
transposed product with and without the weight gradients beside it, and both sides of the lines."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_block import compare_block, inputs
from test_gpu_padded import test_padded_forward as check_padded
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 7, 7, 512, 16, 7, 5),        # 49 rows, one token per region
    (1, 3, 5, 256, 8, 1, 1),         # 15 rows, one region: one step per wavefront
    (2, 6, 9, 320, 10, 3, 2),        # regions of 6, ten steps for eight wavefronts
    (1, 14, 14, 384, 12, 7, 9),      # 12 steps
    (1, 16, 16, 768, 12, 4, 3),      # 16 tokens
    (1, 21, 12, 448, 7, 3, 2),       # 28
    (1, 32, 8, 256, 8, 4, 2),        # 16
    (1, 12, 24, 256, 8, 3, 2),       # 32: 216 workgroups
    (1, 32, 16, 256, 8, 4, 2),       # 384: the other kernel
    (1, 36, 16, 256, 8, 4, 2),       # 36 tokens: too
    (4, 10, 10, 256, 8, 5, 2),       # 312 for Q, K and V, 208 for Q and K: the other kernel for both
    (1, 10, 10, 1088, 17, 5, 2),     # 34 steps
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_forward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9920 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")


@pytest.mark.parametrize("B,H,W,C,heads,S,k,e", [
    (2, 8, 8, 768, 12, 8, 5, 3),
    (1, 3, 5, 384, 12, 1, 1, 1),
    (1, 14, 14, 384, 12, 7, 6, 4),
    (4, 14, 14, 512, 16, 7, 6, 3),
])
def test_block(B, H, W, C, heads, S, k, e):
    X, P = inputs(B, H, W, C, seed=9921 + H * W + C, expansion=e)
    compare_block(X, P, S, k, heads)


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (1, 7, 7, 512, 16, 7, 1),
    (1, 3, 5, 256, 8, 1, 1),
    (2, 7, 7, 768, 24, 7, 2),
    (2, 14, 14, 768, 24, 7, 2),
    (2, 14, 14, 256, 8, 7, 2),
    (3, 6, 9, 320, 10, 3, 2),
])
def test_backward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9922 + H * W + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (1, 13, 12, 384, 12, 7, 4),      # means, zero rows
    (1, 5, 9, 512, 16, 4, 3),        # regions of padding only
    (2, 10, 11, 256, 8, 3, 2),
])
def test_padded(B, H, W, C, heads, S, k):
    check_padded("bf16", B, H, W, C, heads, S, k, "mfma")
