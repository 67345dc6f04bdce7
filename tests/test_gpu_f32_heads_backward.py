"""GPU parity of the float32 gradients where wavefronts share a head of a region (at most 32 tokens, heads of at most 32
channels): four, two and one per head on both sides of the lines between them, fewer heads than a workgroup has places for, one
and two tiles of tokens, one tile of keys and up to more than a wavefront keeps, channels that loads of four do not fit."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward

pytestmark = pytest.mark.gpu

SHAPES = [  # (dtype, B, H, W, C, heads, S, k)
    ("f32", 4, 28, 28, 96, 3, 7, 4),       # 588 heads of regions: four wavefronts each
    ("f32", 25, 8, 16, 48, 3, 4, 3),       # 1200: two
    ("f32", 26, 8, 16, 48, 3, 4, 3),       # 1248: one on the query side, two on the key side
    ("f32", 50, 8, 8, 32, 2, 4, 2),        # 1600: two heads, two wavefronts
    ("f32", 51, 8, 8, 32, 2, 4, 2),        # 1632
    ("f32", 40, 12, 12, 96, 3, 4, 5),      # 1920: one
    ("f32", 60, 12, 12, 32, 1, 4, 2),      # one head: four, however many
    ("f32", 2, 16, 16, 160, 5, 4, 4),      # five heads
    ("f32", 1, 14, 14, 64, 2, 7, 49),      # 13 tiles of keys for four wavefronts
    ("f32", 2, 16, 16, 64, 2, 4, 16),      # 16: the most that are kept
    ("f32", 2, 16, 17, 64, 2, 1, 1),       # 272 tokens per region: not by heads
    ("f32", 1, 20, 20, 64, 2, 4, 11),      # 25 tokens: two tiles, 18 tiles of keys
    ("f32", 3, 16, 32, 64, 2, 4, 4),       # 32 tokens, 8 tiles of keys
    ("f32", 3, 16, 16, 64, 2, 4, 2),       # 16 tokens
    ("f32", 3, 17 * 2, 2, 64, 2, 2, 1),    # 17 tokens
    ("f32", 3, 33 * 2, 2, 64, 2, 2, 1),    # 33
    ("f32", 2, 12, 12, 60, 6, 3, 3),       # heads of 10 channels
    ("f32", 70, 6, 9, 30, 5, 3, 2),        # of 6, one wavefront per head
    ("bf16", 2, 12, 20, 72, 3, 4, 5),      # of 24
    ("bf16", 5, 14, 28, 96, 3, 7, 12),
    # lists of 4, 12, 16 and 64 rows on average: one, one, two and four wavefronts on the key side
    ("f32", 2, 14, 14, 256, 8, 7, 1),
    ("f32", 4, 14, 14, 96, 3, 7, 3),
    ("f32", 4, 14, 14, 96, 3, 7, 4),
    ("f32", 4, 14, 14, 96, 3, 7, 16),
    # as many wavefronts as keep the weights: 4, 5, 8, 9, 16 and 17 tiles of keys at more than 1200 heads of regions
    ("f32", 7, 14, 28, 128, 4, 7, 8),
    ("f32", 7, 14, 28, 128, 4, 7, 9),
    ("f32", 7, 14, 28, 128, 4, 7, 16),
    ("f32", 7, 14, 28, 128, 4, 7, 17),
    ("f32", 7, 14, 28, 128, 4, 7, 32),
    ("f32", 7, 14, 28, 128, 4, 7, 33),
    ("f32", 11, 21, 42, 96, 3, 7, 4),      # 18 tokens, 5 tiles: two
    # heads of 10 channels, four wavefronts, with one and with two tiles of tokens; two on the query side and on both; one, in loads of four too
    ("f32", 2, 12, 12, 30, 3, 3, 4),
    ("f32", 2, 15, 15, 30, 3, 3, 3),
    ("f32", 2, 15, 15, 30, 3, 3, 1),
    ("f32", 2, 9, 18, 30, 3, 3, 1),
    ("f32", 60, 9, 18, 30, 3, 3, 1),
    ("f32", 60, 9, 18, 96, 3, 3, 1),
    # 17 to 32 tokens: one block of 33 to 64 keys, of two heads to a workgroup; 32 keys and 66
    ("f32", 2, 12, 10, 64, 2, 2, 2),       # 30 tokens, 60 keys
    ("f32", 3, 16, 32, 160, 5, 4, 2),      # 64 keys, an odd number of heads
    ("f32", 2, 15, 15, 60, 6, 3, 2),       # heads of 10 channels
    ("f32", 2, 16, 32, 64, 2, 4, 1),
    ("f32", 3, 24, 12, 96, 3, 4, 4),       # 72 keys
    ("f32", 2, 12, 10, 32, 1, 2, 2),       # one head
    ("bf16", 2, 35, 35, 96, 3, 7, 2),
]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", SHAPES)
def test_heads_backward(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9950 + H * W + C + k, dtype=dtype)
    compare_backward(X, Wqkv, Wo, Wlce, dtype, heads, S, k, path="generic")
