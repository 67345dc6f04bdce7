"""GPU parity of the general pipeline's attention with the output projection behind it (64 channels, two heads): a head of one or of two
query tiles per wavefront and both heads, keys by division and by walking, ragged query tiles, wavefronts without queries, maps
that are padded."""
import pytest
import torch

import oracle
import paper_2303_08810_amd as bra
from parity_util import check_output, check_routing, to_device, to_numpy
from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, k), 16 x 16 regions
    (1, 48, 176, 4),         # 33 tokens: a query tile of one, a wavefront without any
    (1, 80, 112, 9),         # 35 tokens, 315 keys
    (4, 80, 112, 1),         # 1024 workgroups: both heads per wavefront
    (4, 80, 112, 6),
    (2, 128, 256, 1),        # 128 tokens, 512 workgroups of two query tiles per wavefront
    (2, 112, 272, 2),        # 119 tokens
    (3, 112, 272, 1),        # 768 workgroups: both heads of two query tiles
    (8, 96, 176, 4),         # 66 tokens, 2048 workgroups: the same, keys by walking
]


@pytest.mark.parametrize("B,H,W,k", SHAPES)
def test_attention_out(B, H, W, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, 64, seed=7800 + H + W + k, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", 16, k, 2, "mfma", images=[B - 1])


PADDED = [  # (B, H, W, S, k)
    (1, 75, 110, 16, 3),     # 5 x 7 tokens, the last rows and columns beyond the map
    (2, 113, 260, 16, 1),    # 8 x 17
    (2, 121, 255, 16, 2),    # 8 x 16, two query tiles per wavefront
    (3, 113, 260, 16, 1),    # both heads of two
]


@pytest.mark.parametrize("B,H,W,S,k", PADDED)
def test_attention_out_padded(B, H, W, S, k):
    arrays = make_inputs(B, H, W, 64, seed=7850 + H + W + k, dtype="bf16")
    X, Wqkv, Wo, Wlce = (to_device(a, "bf16") for a in arrays)
    Y, Ir = bra.bra_forward_padded(X, Wqkv, Wo, Wlce, S, k, 2, want_Ir=True)
    torch.cuda.synchronize()
    Ir = Ir.cpu().numpy()
    check_routing(Ir, oracle.bra_forward_padded(*arrays, S=S, k=k, heads=2, threads=8)["Ar"], k)
    ref = oracle.bra_forward_padded(*arrays, S=S, k=k, heads=2, threads=8, Ir_in=Ir)
    check_output(to_numpy(Y), ref["Y"], "bf16")
