"""GPU parity of the general pipeline's depth-wise convolution where the height of its strips changes: one strip of 24 rows,
two of 13 and 12, low strips where every block has a compute unit beside the choice of regions, high ones where not; and of the gradient's passes."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

STRIPS = [  # (B, H, W, C, heads, S, k)
    (1, 3, 3, 64, 1, 1, 1),
    (64, 24, 24, 64, 1, 2, 1),       # 24 rows, beside 64 blocks or more
    (1, 25, 5, 64, 2, 5, 25),        # 7 x 4 rows at most, alone
    (40, 25, 45, 64, 1, 5, 1),       # two strips, the lower one a row short
    (8, 32, 32, 768, 12, 2, 2),      # 16 rows: the lowest that leave each block alone
    (2, 34, 18, 192, 6, 2, 4),
    (3, 50, 7, 192, 3, 1, 1),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", STRIPS)
def test_lce_strips(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=7600 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1])


GRADIENT = [  # (B, H, W, C, heads, S, k): even strips of the two passes
    (64, 14, 14, 384, 12, 7, 4),     # one strip of 14 rows
    (3, 21, 10, 64, 1, 1, 1),        # five of 5 and 1
    (16, 28, 28, 192, 6, 7, 1),      # four of 7
    (32, 41, 36, 64, 2, 1, 1),       # three of 14 and 13
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", GRADIENT)
def test_gradient_strips(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=7650 + H * W + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
