"""GPU parity of the general pipeline's products at the sizes that pick each tile (128 x 128, 64 x 128, 64 x 64), with
ragged rows, a last column tile that is not full and an odd number of 64-deep chunks, with and without the
region-level projection in the same launch."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

EDGES = [  # (B, H, W, C, heads, S, k)
    (200, 7, 7, 448, 14, 7, 5),      # 128 x 128 tiles (77 row tiles, 10.5 column tiles), K = 7 chunks
    (50, 14, 14, 448, 14, 7, 5),     # the same with 2450 region rows
    (90, 7, 7, 320, 10, 7, 3),       # 64 x 128 tiles, K = 5 chunks
    (36, 14, 14, 320, 10, 7, 3),     # the same with 1764 region rows
    (3, 14, 14, 192, 6, 7, 4),       # 64 x 64 tiles
    (1, 3, 3, 64, 1, 3, 2),          # 9 rows, one chunk
    (15, 18, 18, 1024, 32, 2, 2),    # weights of 6 MB, 4860 rows, with region rows (81 tokens each)
    (20, 14, 14, 192, 6, 7, 3),      # W^o: 3920 rows of one and a half tiles of columns
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", EDGES)
def test_gemm_tiles(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8500 + B + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1] if B > 1 else None)


ROWS = [  # (B, H, W, C, heads, S, k): one wavefront per region and 64 channels: query tiles of 16 and 32, ragged key blocks,
          # several 32-key blocks, idle wavefronts in the last group, two heads of 32 or one of 64 per wavefront
    (2, 12, 12, 192, 3, 3, 2),       # n = 16, 32 keys: one block
    (1, 15, 9, 320, 5, 3, 3),        # n = 15, 45 keys, five groups of 64 channels
    (1, 12, 15, 384, 12, 3, 5),      # n = 20, 100 keys, heads of 32
    (2, 8, 16, 64, 1, 2, 3),         # n = 32, 96 keys
    (1, 22, 6, 192, 6, 2, 1),        # n = 33: the 64-query kernel
    (1, 6, 6, 512, 8, 6, 36),        # n = 1, heads of 64, 36 keys
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", ROWS)
def test_attention_rows(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8700 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")


TILES = [  # the kernel for larger regions: one and two query tiles per wavefront, ragged query tiles and key blocks, growing
           # scores (the softmax reference has to move after the first block)
    (1, 20, 20, 192, 6, 4, 3),       # n = 25: the small-region kernel, for comparison
    (1, 24, 28, 192, 6, 4, 5),       # n = 42, 210 keys
    (2, 16, 64, 64, 1, 2, 3),        # n = 256, heads of 64
    (64, 26, 38, 64, 2, 2, 4),       # n = 247: 128-query tiles, 988 keys (images 0 and 63 compared)
    (11, 77, 77, 64, 2, 7, 1),       # n = 121: 128-query tiles, 121 keys, rows by divisions
    (1, 104, 152, 64, 2, 8, 4),      # n = 247: 256 of 256 queries in two 128-query tiles, 988 keys
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", TILES)
def test_attention_large_regions(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8600 + H * W + C, dtype="bf16")
    images = [0, B - 1] if B > 2 else None
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=images)
    if B <= 2:
        compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", scale=0.5)


@pytest.mark.parametrize("C", [64, 128])
def test_many_rows(C):
    # W in LDS, wavefronts walking over row tiles: 40817 and 100842 rows (the last tile with 1 and 10), Q | K | V, the region
    # rows in a launch of their own, dO by the transposed product
    X, Wqkv, Wo, Wlce = make_inputs(42, 49, 49, C, seed=9800 + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", 7, 2, C // 32, "mfma", images=[0, 41])
    X = X[:17]
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", C // 32, 7, 1, path="mfma")
