"""GPU parity on both sides of the lines between the pipelines of small regions: image-resident attention from 256 (image,
head) pairs on, a wavefront per region below; more than 64 regions; and the routing on its own, which has to give the index of
the forward pass."""
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import to_device
from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (31, 14, 14, 256, 8, 7, 16),     # 248 pairs
    (32, 14, 14, 256, 8, 7, 16),     # 256
    (63, 14, 14, 128, 4, 7, 16),     # 252
    (64, 14, 14, 128, 4, 7, 16),     # 256
    (64, 14, 28, 128, 4, 7, 4),      # 8 tokens per region
    (16, 14, 14, 512, 16, 7, 15),    # 256 pairs, 12544 blocks of keys
    (16, 14, 14, 512, 16, 7, 8),     # 6272
    (48, 7, 7, 192, 6, 7, 3),        # 288 pairs, 192 workgroups of the routing
    (1, 64, 64, 64, 2, 16, 4),       # 256 regions of 16 tokens
    (1, 72, 72, 128, 4, 9, 2),       # 81 of 64
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_lines(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9500 + B + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1] if B > 1 else None)
    Xd, Wd, Wod, Wld = (to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce))
    Y, Ir = bra.bra_forward(Xd, Wd, Wod, Wld, S, k, heads, want_Ir=True, path="mfma")
    assert torch.equal(Ir, bra.bra_route(Xd, Wd, S, k, heads, path="mfma"))
