"""GPU parity of the float32 family at the edges of its tiles: query tiles of 16 / 32 / 64 tokens, key blocks of
32 / 64, heads that are not multiples of 4 channels (scalar loads) or of a head group, odd channel counts,
product tiles with ragged rows, columns and contraction, strips of the depth-wise gradients, and more routing
entries than one list chunk of the key side holds."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

EDGES = [  # (B, H, W, C, heads, S, k)
    (1, 8, 8, 96, 3, 2, 2),          # n = 16, three heads in a group of four, 32 keys: one key block exactly
    (2, 6, 22, 60, 3, 2, 1),         # n = 33, heads of 20 channels, 33 keys
    (1, 21, 13, 66, 3, 1, 1),        # one region of 273 tokens, heads of 22 channels, five key blocks
    (1, 10, 10, 65, 5, 5, 8),        # odd channel count, heads of 13, n = 4, 32 keys
    (3, 9, 12, 64, 1, 3, 5),         # one head of 64, n = 12
    (1, 16, 32, 40, 2, 16, 5),       # 1280 routing entries per image: two list chunks
    (1, 26, 8, 128, 2, 2, 4),        # n = 52, heads of 64, 208 keys
    (1, 14, 20, 40, 2, 2, 3),        # n = 70: five query tiles in one workgroup
    (1, 18, 20, 128, 2, 2, 2),       # n = 90, heads of 64: six
    (1, 5, 7, 4, 1, 1, 1),           # C = 4: one 4-channel chunk
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", EDGES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_f32_family_edges(B, H, W, C, heads, S, k, dtype):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=7000 + H * W + C + k, dtype=dtype)
    compare(X, Wqkv, Wo, Wlce, dtype, S, k, heads, "generic")
    compare_backward(X, Wqkv, Wo, Wlce, dtype, heads, S, k, path="generic")


ROUTES = [  # (B, H, W, C, heads, S, k): region counts around the row tile and the key groups, channel slices 1 .. 8
    (1, 5, 5, 16, 1, 5, 25),         # 25 regions, one channel step
    (2, 9, 9, 24, 1, 9, 40),         # 81 regions: two key groups, k beyond the small ranking
    (1, 16, 16, 192, 6, 16, 3),      # 256 regions, eight slices
    (1, 17, 17, 33, 1, 17, 5),       # 289 regions, scalar loads
    (1, 32, 32, 32, 1, 32, 2),       # 1024 regions
    (3, 8, 8, 320, 10, 8, 64),       # k = all of 64 regions
    (1, 1, 1, 64, 2, 1, 1),          # one region
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", ROUTES)
def test_routing_rows_edges(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=7500 + S + C, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, heads, "generic")
