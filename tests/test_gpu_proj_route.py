"""GPU parity of the layers of 64 channels whose projection carries the routing from pooled X: one tile per wavefront, workgroups that are not full,
several tiles per wavefront and a ragged last workgroup."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 16, 8, 64, 2, 1, 1),         # one region
    (1, 16, 24, 64, 2, 2, 2),        # 24 tiles
    (3, 40, 40, 64, 2, 5, 3),        # 300
    (3, 112, 112, 64, 2, 7, 2),      # 2352: two per wavefront
    (9, 112, 112, 64, 2, 7, 2),      # 7056: four, the last workgroup with one tile
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_projection_with_routing(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9940 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=sorted({0, B - 1}))
