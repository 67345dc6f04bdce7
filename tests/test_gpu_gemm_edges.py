"""GPU parity of the general pipeline's products at the sizes that pick each tile (128 x 128, 64 x 128, 64 x 64), with
ragged rows, a last column tile that is not full and an odd number of 64-deep chunks, with and without the
region-level projection in the same launch."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

EDGES = [  # (B, H, W, C, heads, S, k)
    (200, 7, 7, 448, 14, 7, 5),      # 128 x 128 tiles (77 row tiles, 10.5 column tiles), K = 7 chunks
    (50, 14, 14, 448, 14, 7, 5),     # the same with 2450 region rows
    (90, 7, 7, 320, 10, 7, 3),       # 64 x 128 tiles, K = 5 chunks
    (23, 14, 14, 320, 10, 7, 3),     # the same with region rows
    (3, 14, 14, 192, 6, 7, 4),       # 64 x 64 tiles
    (1, 3, 3, 64, 1, 3, 2),          # 9 rows, one chunk
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", EDGES)
def test_gemm_tiles(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=8500 + B + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1] if B > 1 else None)
