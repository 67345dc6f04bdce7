"""GPU parity of the layers of 64 channels whose projection carries the routing from pooled X: up to one tile of 16 tokens per wavefront of the launch
(k_qkv), two and four (k_proj_route), workgroups that are not full and a ragged last one."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 16, 8, 64, 2, 1, 1),         # one region
    (1, 16, 24, 64, 2, 2, 2),        # 24 tiles
    (3, 40, 40, 64, 2, 5, 3),        # 300
    (1, 128, 256, 64, 2, 8, 2),      # 2048: one for each
    (1, 128, 264, 64, 2, 8, 2),      # 2112
    (3, 112, 112, 64, 2, 7, 2),      # 2352: two per wavefront
    (9, 112, 112, 64, 2, 7, 2),      # 7056: four, the last workgroup with one tile
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_projection_with_routing(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9940 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=sorted({0, B - 1}))
