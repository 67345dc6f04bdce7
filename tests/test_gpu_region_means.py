"""GPU parity of the region means that come out of the token projection: every way a tile adds up its rows (whole regions of 4
and 16 tokens, groups of 16 or 4 of larger ones, odd counts row by row), idle rows of a tile, a last tile that is not full,
regions of several images in one tile, tiles of 64 and 128 rows and columns, and both sides of the lines beyond which the
means of the tokens are projected."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from synthetic_inputs import make_inputs
from test_gpu_parity import compare
from parity_util import to_device

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (3, 3, 6, 64, 2, 3, 9),          # 2 tokens per region, 27 regions of three images in one tile
    (5, 9, 3, 192, 6, 3, 2),         # 3
    (2, 14, 14, 384, 12, 7, 16),     # 4: whole groups
    (7, 10, 10, 128, 4, 5, 7),       # 4
    (3, 7, 35, 192, 6, 7, 4),        # 5
    (2, 14, 21, 256, 4, 7, 3),       # 6
    (6, 12, 6, 320, 5, 3, 9),        # 8: two groups of 4
    (1, 9, 12, 192, 6, 3, 3),        # 12
    (40, 16, 16, 128, 2, 4, 4),      # 16
    (3, 15, 15, 192, 3, 3, 5),       # 25
    (2, 8, 28, 384, 6, 2, 3),        # 56: one region in a tile of 64 rows, two in one of 128
    (1, 12, 32, 192, 6, 2, 2),       # 96: beyond what a tile of 64 rows holds
    (3, 33, 2, 192, 6, 1, 1),        # 66
    (2, 16, 16, 64, 1, 2, 2),        # 64 tokens, a single chunk of the contraction
    (9, 6, 24, 64, 1, 3, 4),         # 16
    (9, 9, 9, 64, 2, 3, 4),          # 9
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_means_from_the_projection(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9810 + H + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")


# On both sides of the lines, by values in units of 2^20 and tokens per region: 8 tokens at 1024 channels 5.5, 64 4, 6 at 384 8, 16 5, 42 2; 4
# have none
LINES = [(11, 32, 16, 1024, 8, 3), (12, 32, 16, 1024, 8, 3), (21, 32, 32, 192, 4, 2), (22, 32, 32, 192, 4, 2), (56, 16, 24, 384, 8, 3), (57, 16, 24, 384, 8, 3),
         (34, 28, 28, 192, 7, 3), (35, 28, 28, 192, 7, 3), (3, 49, 42, 320, 7, 3), (4, 49, 42, 320, 7, 3),
         (28, 14, 14, 384, 7, 3), (130, 14, 14, 384, 7, 3), (64, 14, 14, 512, 7, 3), (64, 14, 14, 768, 7, 9)]


@pytest.mark.parametrize("B,H,W,C,S,k", LINES)
def test_both_sides_of_the_lines(B, H, W, C, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9840 + B, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, C // 32, "mfma", images=[0, B - 1])


F32 = [  # (dtype, B, H, W, C, heads, S, k): float32 kernels, which take odd multiples of 4 channels too
    ("f32", 5, 7, 7, 64, 2, 7, 9),        # one token per region
    ("f32", 3, 6, 3, 100, 2, 3, 4),       # 2, columns beyond the last tile
    ("f32", 2, 14, 14, 96, 3, 7, 5),      # 4
    ("f32", 2, 9, 9, 36, 1, 3, 3),        # 9
    ("f32", 3, 16, 16, 64, 1, 4, 4),      # 16
    ("f32", 1, 15, 12, 128, 4, 3, 2),     # 20
    ("f32", 2, 16, 12, 192, 6, 2, 3),     # 48
    ("f32", 1, 24, 24, 64, 2, 3, 4),      # 64
    ("f32", 1, 26, 14, 64, 2, 2, 2),      # 91: beyond a tile
    ("bf16", 2, 14, 14, 96, 3, 7, 5),
    ("bf16", 40, 28, 28, 96, 3, 7, 4),    # tiles of 128 columns
    ("bf16", 3, 9, 12, 160, 5, 3, 3),     # 12
    ("bf16", 2, 15, 15, 100, 2, 3, 3),    # 25
]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", F32)
def test_means_of_the_float32_kernels(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9870 + H + C, dtype=dtype)
    compare(X, Wqkv, Wo, Wlce, dtype, S, k, heads, "generic", images=[0, B - 1] if B > 1 else None)


def test_an_infinity_stays_in_its_region():
    """Regions of 12 tokens share tiles and groups of rows are added up across lanes: only the affinities of the region that
    holds the infinity are not finite."""
    B, S, C, heads, k = 2, 4, 192, 6, 3
    X, Wqkv, _, _ = make_inputs(B, 12, 16, C, seed=9850, dtype="bf16")
    X[1, 4, 9, 0] = np.inf           # region 6 of the second image
    _, Ar = bra.bra_route(to_device(X, "bf16"), to_device(Wqkv, "bf16"), S, k, heads, want_Ar=True)
    bad = ~torch.isfinite(Ar.float().cpu())
    want = torch.zeros_like(bad)
    want[1, 6, :] = want[1, :, 6] = True
    assert torch.equal(bad, want)
