"""GPU parity of the float32 family's block where lanes take four channels of a token: one to four steps of them, idle lanes, several tokens to a
wavefront and a ragged last workgroup, more than one token per group, and the kernel for channel counts that four does not divide."""
import pytest

from test_gpu_block import compare_block, inputs

pytestmark = pytest.mark.gpu

SHAPES = [  # (dtype, B, H, W, C, heads, S, k)
    ("f32", 1, 5, 7, 4, 1, 1, 1),
    ("f32", 3, 1, 9, 20, 2, 1, 1),       # five of eight lanes
    ("bf16", 2, 9, 1, 36, 3, 1, 1),
    ("f32", 2, 6, 6, 260, 4, 3, 2),      # two steps, one lane in the second
    ("f32", 1, 4, 6, 768, 12, 2, 1),     # three
    ("f32", 1, 4, 4, 1024, 16, 2, 1),    # four
    ("f32", 1, 2, 4, 1056, 33, 2, 1),    # five: the other kernel
    ("f32", 1, 4, 6, 30, 2, 2, 1),
    ("bf16", 1, 4, 6, 30, 2, 2, 1),
    ("bf16", 42, 28, 28, 96, 3, 7, 1),   # two tokens per group
    ("f32", 42, 28, 28, 96, 3, 7, 1),
]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", SHAPES)
def test_token_ln(dtype, B, H, W, C, heads, S, k):
    X, P = inputs(B, H, W, C, seed=9990 + H * W + C, expansion=1, dtype=dtype)
    compare_block(X, P, S, k, heads, path="generic", images=[0, B - 1], dtype=dtype)
