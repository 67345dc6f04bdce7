"""bra_route gives the very index that bra_forward uses, for every pipeline: both run the same arithmetic, so not even a
tie that only roundings decide may come out differently."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import to_device
from synthetic_inputs import make_inputs

pytestmark = pytest.mark.gpu

# One token per region (every sum is then the projection's own) at the sizes of its tiles; the other pipelines
SHAPES = [  # (dtype, B, H, W, C, heads, S, k)
    ("bf16", 200, 7, 7, 512, 16, 7, 49),
    ("bf16", 100, 7, 7, 64, 2, 7, 49),
    ("bf16", 4, 7, 7, 128, 4, 7, 49),
    ("bf16", 6, 16, 16, 192, 6, 16, 256),
    ("bf16", 64, 14, 14, 384, 12, 7, 49),      # regions of 4 tokens, means projected in the token projection's launch
    ("bf16", 16, 32, 32, 768, 12, 8, 64),
    ("bf16", 8, 52, 76, 64, 2, 4, 16),
    ("bf16", 2, 96, 64, 64, 2, 16, 256),
    ("bf16", 32, 56, 56, 64, 2, 7, 1),         # the specialised pipelines
    ("bf16", 32, 28, 28, 128, 4, 7, 49),
    ("bf16", 32, 14, 14, 256, 8, 7, 49),
    ("bf16", 2, 128, 128, 64, 2, 8, 64),
    ("bf16", 16, 28, 28, 96, 3, 7, 49),        # the float32 family
    ("f32", 16, 28, 28, 64, 2, 7, 4),
    ("f32", 16, 21, 14, 64, 2, 7, 49),
]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", SHAPES)
def test_route_matches_forward(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9700 + C + H, dtype=dtype)
    # the halves of the channels have the same weights, and regions 2 r and 2 r + 1 the same tokens with the halves exchanged:
    # their affinities are equal and differ by the order of summation alone
    Wqkv[C // 2:] = Wqkv[:C // 2]
    V = X.reshape(B, S, H // S, S, W // S, C).transpose(0, 1, 3, 2, 4, 5).reshape(B, S * S, -1, C).copy()
    pairs = S * S // 2
    V[:, 1:2 * pairs:2] = np.roll(V[:, 0:2 * pairs:2], C // 2, axis=-1)
    X = V.reshape(B, S, S, H // S, W // S, C).transpose(0, 1, 3, 2, 4, 5).reshape(B, H, W, C)
    X, Wqkv, Wo, Wlce = (to_device(np.ascontiguousarray(a), dtype) for a in (X, Wqkv, Wo, Wlce))
    Ir = bra.bra_route(X, Wqkv, S, k, heads)
    used = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, heads, want_Ir=True)[1]
    assert torch.equal(Ir, used), f"{int((Ir != used).sum())} of {Ir.numel()} entries differ"
