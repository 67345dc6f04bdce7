"""GPU parity of the attention over regions of more than 32 tokens, by what a wavefront holds: one or both heads of a channel group, of one
or of two query tiles; edges of the query tiles, wavefronts without queries, the fewest workgroups at
which the choice turns."""
import pytest

from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 6, 22, 192, 6, 2, 4),        # 33 tokens: a wavefront with one query, one without
    (1, 16, 20, 192, 6, 2, 1),       # 80 tokens, one tile of keys and a quarter
    (341, 5, 7, 192, 6, 1, 1),       # 35 tokens, 1023 workgroups
    (342, 5, 7, 192, 6, 1, 1),       # 1026
    (171, 8, 16, 192, 6, 1, 1),      # 128 tokens, 513 workgroups of two query tiles
    (170, 8, 16, 192, 6, 1, 1),      # 510: one query tile
    (172, 7, 17, 192, 6, 1, 1),      # 119 tokens: the last wavefront's second tile has 7 queries
    (255, 8, 16, 192, 6, 1, 1),      # 765 workgroups of two query tiles, two blocks of keys
    (256, 7, 17, 192, 6, 1, 1),      # 768: both heads
    (64, 16, 24, 192, 6, 2, 2),      # 96 tokens, 192 keys
    (64, 16, 24, 192, 6, 2, 3),      # 288 keys: a head
    (171, 16, 24, 192, 6, 2, 3),     # 2052 workgroups: both, keys by walking
    (76, 24, 48, 192, 6, 3, 4),      # 512 keys
    (76, 24, 48, 192, 6, 3, 5),      # 640: a head
    (64, 16, 24, 192, 3, 2, 2),      # heads of 64 channels
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_heads_of_a_wavefront(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9730 + B + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1] if B > 2 else None)
