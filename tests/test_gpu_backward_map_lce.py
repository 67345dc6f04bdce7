"""GPU parity of the gradients of images whose slices lie in LDS whole, where the depth-wise parts come from the same slices: 8 and 16 wavefronts,
one pair of items for each and others that take the tap gradients, sides that whole items of 4 x 4 tokens do not fill, more chunks of a row than two
per thread, and one item more than the wavefronts hold (the passes of their own).  An infinity of dO reaches the taps that meet it and no others."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import to_device
from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k)
    (80, 14, 14, 64, 2, 7, 2),       # 16 wavefronts, 8 pairs of items
    (130, 14, 14, 64, 2, 7, 3),      # 8 wavefronts, 8 pairs
    (27, 14, 14, 192, 6, 7, 2),
    (130, 7, 7, 64, 2, 7, 3),        # 2 pairs
    (130, 10, 15, 64, 2, 5, 2),      # 6 pairs
    (130, 13, 13, 64, 2, 13, 2),
    (130, 9, 9, 64, 2, 9, 4),        # 9 items
    (130, 4, 6, 64, 2, 2, 2),        # one strip, the second item with two columns of its own
    (130, 2, 6, 64, 2, 2, 2),        # lower than an item: the passes of their own
    (80, 9, 36, 64, 2, 9, 2),        # 14 pairs of 27 items
    (80, 28, 14, 64, 2, 7, 2),       # 8 tokens per region
    (80, 9, 45, 64, 2, 9, 2),        # 36 items
    # (image, head) pairs beyond which the passes are their own again: 768 with 9 items, 1024 with 4, 256 with 27 and a compute unit for each workgroup
    (96, 12, 12, 256, 8, 6, 2),
    (97, 12, 12, 256, 8, 6, 2),
    (128, 5, 5, 256, 8, 5, 2),
    (129, 5, 5, 256, 8, 5, 2),
    (32, 9, 36, 256, 8, 9, 2),
    (33, 9, 36, 256, 8, 9, 2),
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_slice_convolution(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9970 + H * W + C + k, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", heads, S, k, path="mfma")


# The last token of an image: taps of later rows and columns never meet it
@pytest.mark.parametrize("B,H,W,S", [(80, 14, 14, 7), (130, 7, 7, 7), (130, 10, 15, 5), (130, 13, 13, 13)])
def test_infinity_reaches_the_taps_that_meet_it(B, H, W, S, channel=5):
    C = 64
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9980 + H, dtype="bf16")
    dY = np.asarray(X) * np.float32(0.5)
    dY[1, H - 1, W - 1, 9] = 2.0 ** 100
    Wo[:, 9] = 0
    Wo[channel, 9] = 2.0 ** 40
    Ir = torch.arange(2, dtype=torch.int32).repeat(B, S * S, 1).cuda()
    args = [to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce)]
    taps = bra.bra_backward(*args, Ir, to_device(dY, "bf16"), S, 2, path="mfma")[3].cpu().numpy().reshape(C, 5, 5)
    other = np.arange(C) != channel
    assert np.isfinite(taps[other]).all() and not np.isfinite(taps[channel, :3, :3]).any()
    assert np.isfinite(taps[channel, 3:]).all() and np.isfinite(taps[channel, :, 3:]).all()
