"""GPU parity of the depth-wise kernels on bf16 maps (general pipeline forward, backward) at the edges of their
tiling: one and two columns, odd widths, fewer column pairs than a workgroup's slots (strips above each other), strip
heights 5, 10 and 20 with ragged ends, several tiles per workgroup."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

EDGES = [  # (B, H, W, C, heads, S, k)
    (1, 9, 1, 192, 6, 1, 1),
    (2, 23, 2, 64, 1, 1, 1),
    (1, 22, 5, 128, 2, 1, 1),
    (3, 6, 21, 192, 3, 3, 4),
    (1, 41, 17, 64, 1, 1, 1),
    (40, 20, 36, 64, 1, 2, 1),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", EDGES)
def test_lce_edges(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8000 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1])
    compare_backward(X[:2], Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
    if B > 2:
        compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")


MAPS = [  # (B, H, W, C, heads, S, k): image-resident attention backward: 1 .. 8 tokens per region, one and several key blocks
    (64, 7, 7, 64, 2, 7, 49),        # one token per region, 49 keys
    (64, 10, 5, 64, 2, 5, 7),        # 2 x 1 regions
    (64, 9, 6, 64, 2, 3, 9),         # 3 x 2 regions, every region
    (64, 28, 14, 64, 2, 7, 30),      # 8 tokens, 392 tokens per image (16 wavefronts, most of the LDS), 4 key blocks
    (32, 16, 16, 96 + 32, 4, 8, 16), # 64 keys exactly
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", MAPS)
def test_backward_image_resident(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8800 + H * W + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")


REGIONS = [  # (B, H, W, C, heads, S, k): attention backward region by region
    # a wavefront per region: 1, 16, 17 and 32 tokens; one block of keys, ragged blocks, more entries than one list holds
    (2, 7, 7, 64, 1, 7, 33),
    (6, 28, 28, 64, 2, 7, 3),
    (2, 119, 7, 64, 2, 7, 3),
    (2, 32, 64, 192, 6, 8, 16),
    (5, 28, 21, 128, 4, 7, 7),
    # four wavefronts per tile: two blocks, ragged tiles of 32 tokens, five
    (1, 28, 28, 64, 2, 7, 4),
    (2, 10, 14, 64, 1, 2, 3),
    (1, 35, 28, 128, 2, 7, 20),
    # four tiles of a region per workgroup: idle wavefronts, whole tiles, two tiles per wavefront
    (4, 42, 42, 128, 4, 7, 3),
    (3, 56, 56, 128, 2, 7, 1),
    (9, 88, 80, 64, 2, 8, 2),
    (5, 70, 77, 128, 2, 7, 3),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", REGIONS)
def test_backward_regions(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9200 + H * W + C, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")
