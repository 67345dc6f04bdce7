"""bra_route and bra_forward_static give the very index that bra_forward uses, for every pipeline: all run the same arithmetic,
so not even a tie that only roundings decide may come out differently."""
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
    # float32, means of the tokens projected: bra_route's product on its own, bra_forward's beside Q, K and V
    ("f32", 16, 56, 56, 64, 2, 7, 4),          # 64 tokens per region, more tiles than the means come out of
    ("f32", 16, 56, 56, 64, 2, 7, 49),
    ("f32", 1, 128, 128, 64, 2, 8, 4),         # more than 64 tokens
    ("f32", 2, 63, 63, 128, 4, 7, 49),
    ("f32", 2, 63, 63, 192, 6, 7, 49),
    ("f32", 1, 63, 63, 256, 8, 7, 49),
    ("f32", 2, 63, 63, 96, 3, 7, 49),
    # few rows, whose contraction the wavefronts of a workgroup share: means out of the projection, one token per region
    ("f32", 2, 16, 16, 256, 8, 4, 3),
    ("f32", 1, 35, 28, 192, 6, 7, 49),
    ("f32", 1, 7, 7, 512, 16, 7, 49),
    ("bf16", 1, 7, 7, 512, 16, 7, 5),
    ("bf16", 4, 7, 7, 384, 12, 7, 49),
    ("bf16", 1, 14, 14, 384, 12, 7, 9),
    ("bf16", 2, 14, 14, 1024, 32, 7, 49),
    ("bf16", 3, 112, 112, 64, 2, 7, 2),        # 64 channels with all weights in LDS beside the routing
    ("bf16", 10, 64, 64, 64, 2, 8, 64),
]


def paired_inputs(dtype, B, H, W, C, S):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9700 + C + H, dtype=dtype)
    # the halves of the channels have the same weights, and regions 2 r and 2 r + 1 the same tokens with the halves exchanged:
    # their affinities are equal and differ by the order of summation alone
    Wqkv[C // 2:] = Wqkv[:C // 2]
    V = X.reshape(B, S, H // S, S, W // S, C).transpose(0, 1, 3, 2, 4, 5).reshape(B, S * S, -1, C).copy()
    pairs = S * S // 2
    V[:, 1:2 * pairs:2] = np.roll(V[:, 0:2 * pairs:2], C // 2, axis=-1)
    X = V.reshape(B, S, S, H // S, W // S, C).transpose(0, 1, 3, 2, 4, 5).reshape(B, H, W, C)
    return [to_device(np.ascontiguousarray(a), dtype) for a in (X, Wqkv, Wo, Wlce)]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", SHAPES)
def test_route_matches_forward(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = paired_inputs(dtype, B, H, W, C, S)
    Ir = bra.bra_route(X, Wqkv, S, k, heads)
    used = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, heads, want_Ir=True)[1]
    assert torch.equal(Ir, used), f"{int((Ir != used).sum())} of {Ir.numel()} entries differ"


# More than 64 regions, where the pipeline of bra_forward needs more scratch than the built-in buffer has and another one runs
@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (17, 64, 64, 64, 2, 16, 32), (18, 64, 64, 64, 2, 16, 4),        # 16 tokens, 4.5 x 2^20 values: means out of the projection
    (9, 64, 64, 128, 4, 16, 32), (4, 64, 64, 256, 8, 16, 32),
    (4, 128, 128, 64, 2, 16, 8), (2, 128, 128, 128, 4, 16, 8),      # 64 tokens, 4 x 2^20
    (5, 128, 128, 64, 2, 16, 8)])                                   # beyond: means of the tokens, projected
def test_static_matches_forward(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = paired_inputs("bf16", B, H, W, C, S)
    assert bra.workspace_bytes(bra.make_shape(B, H, W, C, heads, S, k, torch.bfloat16)) > bra.STATIC_SCRATCH_BYTES
    used = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, heads, want_Ir=True)[1]
    static = torch.full_like(used, -1)
    bra.bra_forward_static(X, Wqkv, Wo, Wlce, S, k, heads, out=torch.empty_like(X), Ir_out=static)
    assert torch.equal(static, used), f"{int((static != used).sum())} of {used.numel()} entries differ"
    assert torch.equal(bra.bra_route(X, Wqkv, S, k, heads), used)
