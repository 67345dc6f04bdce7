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
    (5, 128, 128, 64, 2, 16, 4),     # 256 of 64
    (6, 128, 128, 64, 2, 16, 4),
    (9, 72, 144, 64, 2, 9, 2),       # 81 of 128
    (10, 64, 64, 128, 4, 16, 5),     # 5 x 2^20 values
    (11, 64, 64, 128, 4, 16, 5),     # above: the layer kernels behind the general pipeline's routing
    (3, 128, 128, 128, 4, 32, 4),    # 1024 of 16
    (56, 64, 64, 64, 2, 16, 4),
    (57, 64, 64, 64, 2, 16, 4),
    (15, 64, 64, 256, 8, 16, 2),
    (16, 14, 14, 512, 16, 7, 9),     # 4 tokens, 36 keys, 256 pairs
    (12, 10, 10, 768, 24, 5, 9),     # 288, 25 regions: 7200 blocks of keys
    (19, 10, 10, 768, 24, 5, 9),     # 11400
    (20, 10, 10, 768, 24, 5, 9),     # 12000
    (39, 10, 10, 768, 24, 5, 8),     # 936 pairs, one block of keys each: 11700
    (40, 10, 10, 768, 24, 5, 8),     # 12000
    (31, 14, 28, 512, 16, 7, 5),     # 8 tokens, 40 keys: 496 pairs, 512 and 528, two rounds and a little more
    (32, 14, 28, 512, 16, 7, 5),
    (33, 14, 28, 512, 16, 7, 5),
    (32, 10, 20, 512, 16, 5, 5),     # two workgroups per compute unit
    (64, 12, 24, 512, 16, 6, 12),    # no room for the convolution: 9 x 2^20 values
    (65, 12, 24, 512, 16, 6, 12),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_lines(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9500 + B + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma", images=[0, B - 1] if B > 1 else None)
    Xd, Wd, Wod, Wld = (to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce))
    Y, Ir = bra.bra_forward(Xd, Wd, Wod, Wld, S, k, heads, want_Ir=True, path="mfma")
    assert torch.equal(Ir, bra.bra_route(Xd, Wd, S, k, heads, path="mfma"))


# The padded map by the general pipeline, the whole one by the layer kernels
@pytest.mark.parametrize("B,H,W,C,heads,S,k", [(22, 127, 126, 64, 2, 16, 4), (12, 63, 60, 128, 4, 16, 4)])
def test_padded_maps_of_many_regions(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = (to_device(a, "bf16") for a in make_inputs(B, H, W, C, seed=9560, dtype="bf16"))
    Y, Ir = bra.bra_forward_padded(X, Wqkv, Wo, Wlce, S, k, heads, want_Ir=True)
    whole = torch.zeros(B, -(-H // S) * S, -(-W // S) * S, C, dtype=X.dtype, device=X.device)
    whole[:, :H, :W] = X
    Y2, Ir2 = bra.bra_forward(whole, Wqkv, Wo, Wlce, S, k, heads, want_Ir=True)
    assert torch.equal(Ir, Ir2)
    # two results with three independent roundings each: sqrt(2) x 2.9e-3 apart
    assert float((Y.double() - Y2[:, :H, :W].double()).norm() / Y2[:, :H, :W].double().norm()) < 5e-3
