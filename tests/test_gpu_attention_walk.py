"""GPU parity of the attention kernels that find their rows by carrying (region, slot) along: steps over several small
regions, regions that no block size divides, the largest slot table and regions beyond it (divisions instead), the second
sweep of the gradients' query side walking back over three blocks and more."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (2, 12, 12, 128, 2, 12, 28),     # one token per region, 28 keys
    (2, 21, 9, 192, 6, 3, 9),        # 21 tokens, 189 keys
    (1, 31, 13, 64, 1, 1, 1),        # 403 tokens in one region
    (1, 45, 95, 192, 6, 5, 7),       # 171 tokens, 1197 keys
    (1, 32, 32, 64, 2, 1, 1),        # 1024 slots
    (1, 41, 25, 64, 2, 1, 1),        # 1025
    (1, 82, 50, 64, 1, 2, 3),        # 1025, three regions
    (1, 32, 32, 64, 2, 2, 4),        # 256 slots, four wavefronts per tile in the gradients
    (1, 20, 52, 64, 1, 2, 2),        # 260
    (2, 24, 24, 64, 1, 3, 3),        # 64 slots, 192 keys: divisions in the forward pass
    (1, 15, 39, 192, 6, 3, 3),       # 65, 195 keys
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_rows_by_walking(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9900 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
