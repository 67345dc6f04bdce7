"""GPU parity of the layers whose image-resident attention forms the convolution of the head's slice in LDS by items of 4 x 4 outputs: maps
narrower and lower than one item, widths and heights that no item divides, fewer items than a workgroup has lane groups and
several rounds of them, regions of 1 to 8 tokens."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (260, 1, 2, 64, 2, 1, 1),        # one item, two columns of it
    (130, 3, 3, 64, 2, 3, 9),        # 3 x 3 map, one token per region
    (65, 7, 7, 128, 4, 7, 49),       # four items
    (40, 5, 10, 256, 8, 5, 7),       # 1 x 2 tokens per region
    (33, 14, 14, 256, 8, 7, 16),     # 16 items, one per lane group
    (33, 21, 42, 256, 8, 21, 3),     # 66 items, 441 regions of 1 x 2
    (22, 20, 10, 768, 24, 5, 12),    # 4 x 2 tokens per region, a ragged last column
    (34, 28, 14, 512, 16, 7, 9),     # 8 tokens per region
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_convolution_in_slices(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9950 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=sorted({0, B // 2, B - 1}))
