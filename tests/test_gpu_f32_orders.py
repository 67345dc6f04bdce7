"""GPU parity of the float32 kernels' attention and its gradients with both orders of workgroups, those of an image and head group on one
XCD and the head groups of a region apart: a number of workgroups that 8 does not divide, one and several query tiles and head
groups, a last head group that is not full, and both sides of each line between the orders; against the oracle and its float32 error bounds."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

FORWARD = [  # (B, H, W, C, heads, S, k)
    (1, 35, 35, 256, 8, 7, 8), (1, 35, 35, 256, 8, 7, 9),      # a sixth of the regions, 196 workgroups
    (1, 15, 9, 160, 5, 3, 9),         # 5 heads in two groups, 18
    (1, 35, 40, 96, 3, 5, 25),        # 56 tokens: a head and four tiles a workgroup, 75
    (2, 9, 12, 192, 3, 3, 5), (2, 9, 12, 192, 3, 3, 6),        # heads of 64 channels; five eighths of the regions
    (3, 9, 9, 128, 4, 3, 9), (4, 9, 9, 128, 4, 3, 9),          # with the output projection
    (2, 15, 15, 384, 12, 3, 9), (1, 15, 15, 512, 16, 3, 9),    # 12 and 8 pairs
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", FORWARD)
def test_forward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9900 + H * W + C, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, heads, "generic")


BACKWARD = [  # (B, H, W, C, heads, S, k)
    (1, 15, 9, 160, 5, 3, 4), (1, 15, 9, 160, 5, 3, 5),        # two head groups, half of the regions
    (1, 35, 40, 96, 3, 5, 3),         # three
    (2, 15, 15, 96, 3, 3, 2),
    (2, 12, 12, 512, 16, 3, 9),       # 8 pairs
    (3, 15, 15, 256, 8, 5, 25),       # 6
    (1, 64, 64, 64, 2, 32, 4),        # 1024 workgroups
    (2, 64, 64, 96, 3, 32, 2),        # 2048
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", BACKWARD)
def test_backward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9930 + H * W + C, dtype="f32")
    compare_backward(X, Wqkv, Wo, Wlce, "f32", heads, S, k, path="generic")
