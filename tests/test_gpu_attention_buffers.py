"""GPU parity of the attention over regions of up to 16 tokens where one buffer of keys per wavefront is enough (more wavefronts than two
workgroups per compute unit hold): two blocks of keys with a ragged and a full last one, three, heads of 64 and of 32 channels, and the
two sides of that line."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (3, 32, 32, 768, 12, 8, 3),      # 2304 wavefronts, 48 keys
    (3, 32, 32, 768, 24, 8, 4),      # 64
    (7, 28, 21, 384, 12, 7, 6),      # 2058, regions of 12 tokens, 72 keys
    (2, 32, 32, 1024, 16, 8, 3),     # 2048: two buffers
    (4, 32, 32, 512, 16, 8, 5),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_one_buffer(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9970 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1])
