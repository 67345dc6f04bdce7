"""GPU parity of float32 layers whose attention carries the output projection (64 channels, two heads, and 128, four): one and two query tiles of a region,
ragged ones, four to six in a workgroup and several workgroups per region, ragged blocks of keys; against the oracle and its float32 error
bounds, and the same index as the routing on its own."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, S, k)
    (48, 14, 14, 7, 5),       # 4 tokens per region
    (31, 28, 21, 7, 3),       # 12 tokens, 36 keys
    (25, 20, 25, 5, 2),       # 20 tokens: a second tile of 4
    (3, 35, 42, 7, 2),        # 30 tokens
    (2, 42, 49, 7, 1),        # 42 tokens: three tiles in four
    (4, 56, 56, 7, 3),        # 64 tokens, three whole blocks of keys
    (11, 45, 40, 5, 2),       # 72 tokens: five tiles in a workgroup
    (2, 45, 40, 5, 1),        # the same in fours
    (14, 60, 35, 5, 1),       # 84 tokens: six tiles
    (36, 32, 32, 2, 1),       # 256 tokens: four workgroups of a region
    (4, 48, 63, 3, 1),        # 336 tokens: six, the last of one tile
    (6, 49, 56, 7, 3), (6, 49, 56, 7, 4),        # 56 tokens, three blocks of keys and four: both sides of the line of three rounds
    (2, 105, 35, 7, 4), (2, 105, 35, 7, 5),      # 75, five and six: of one
]


@pytest.mark.parametrize("B,H,W,S,k", SHAPES)
def test_f32_attention_out(B, H, W, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, 64, seed=7700 + H * W, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, 2, "generic", images=[0, B - 1])


WIDE = [  # (B, H, W, S, k)
    (1, 14, 14, 7, 4),        # 4 tokens per region, half a block of keys
    (24, 14, 14, 7, 16),      # 1176 regions: two blocks of keys
    (25, 14, 14, 7, 5),       # 1225: the products apart
    (3, 21, 21, 7, 11),       # 9 tokens, 99 keys
    (6, 28, 28, 7, 4),        # 16 tokens
    (2, 20, 12, 4, 16),       # 15 tokens, 240 keys
]


@pytest.mark.parametrize("B,H,W,S,k", WIDE)
def test_f32_attention_out_four_heads(B, H, W, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, 128, seed=7760 + H * W, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, 4, "generic", images=[0, B - 1])
