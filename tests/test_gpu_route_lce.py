"""GPU parity where the convolution of V shares the routing's launch and the attention adds itself to it: one tile and odd
numbers of them, several groups of 64 channels, widths and heights that no strip divides, up to 1024 regions, and a given
routing index (the convolution in a launch of its own)."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import check_output, run_oracle, to_device, to_numpy
from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 6, 6, 64, 1, 3, 2),
    (1, 20, 10, 192, 3, 2, 1),
    (3, 10, 50, 64, 1, 5, 3),
    (1, 45, 21, 320, 10, 3, 4),
    (1, 64, 64, 64, 1, 32, 9),       # 1024 regions
    (2, 51, 34, 128, 2, 17, 40),     # 289
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_convolution_beside_routing(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9700 + H * W + C, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [SHAPES[0], SHAPES[2], SHAPES[3]])
def test_convolution_alone(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9750 + H * W + C, dtype="bf16")
    rng = np.random.Generator(np.random.PCG64(9751))
    Ir = np.stack([rng.permutation(S * S)[:k] for _ in range(B * S * S)]).reshape(B, S * S, k).astype(np.int32)
    Y = bra.bra_forward(*(to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce)), S, k, heads, Ir_in=torch.from_numpy(Ir).cuda(), path="mfma")
    check_output(to_numpy(Y), run_oracle(X, Wqkv, Wo, Wlce, dict(S=S, k=k, heads=heads), Ir_in=Ir)["Y"], "bf16")
