"""GPU parity of the weight gradients as partial matrices over shares of the tokens, from C = 128 on: one chunk of 64 tokens and
a part of one, a last share that is shorter than the others, as many shares as two workgroups per compute unit allow and
fewer, dX in the same launch (up to 256 tiles of 128 x 128) and in one of its own."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 4, 4, 128, 4, 4, 2),         # 16 tokens
    (1, 8, 16, 128, 2, 4, 3),        # two whole chunks, a share each
    (3, 12, 12, 128, 4, 4, 3),       # 7 chunks, the last of 48 tokens
    (13, 14, 14, 128, 2, 7, 4),      # 40 chunks in 14 shares of 3, the last of 52 tokens
    (41, 28, 28, 128, 4, 7, 1),      # 252 tiles
    (42, 28, 28, 128, 4, 7, 1),      # 258
    (5, 14, 14, 512, 16, 7, 2),      # 16 chunks in 2 shares, of 8 that would fill the chip
    (2, 7, 7, 1024, 32, 7, 3),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_weight_gradients_over_shares(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9800 + B + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
