"""GPU parity of the attention over small regions with at most 32 routed keys, which keep one block of keys in LDS, and just
beyond: one key, the full block, one key more, groups of regions that do not fill the last workgroup."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 7, 7, 768, 12, 7, 1),        # one key
    (3, 7, 7, 512, 16, 7, 31),
    (1, 6, 6, 64, 1, 6, 32),
    (1, 6, 6, 192, 6, 6, 33),
    (2, 16, 16, 192, 3, 4, 2),       # 16 tokens, 32 keys
    (1, 15, 27, 64, 2, 3, 1),        # 45 tokens: the kernel for larger regions
    (1, 12, 27, 384, 6, 3, 1),       # 36
    (1, 12, 24, 320, 10, 3, 1),      # 32, two query tiles
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_one_block_of_keys(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9650 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")
