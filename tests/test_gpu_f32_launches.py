"""GPU parity of the float32 family where the depth-wise passes share launches with the routing and with the gradients'
attention: one to seven columns, heights that strips of four rows do not divide, channel counts with 4-, 2- and 1-channel
loads, more than 64 channels, and a given routing index (the convolution in a launch of its own)."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import check_output, run_oracle, to_device, to_numpy
from synthetic_inputs import make_inputs
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

SHAPES = [  # (dtype, B, H, W, C, heads, S, k)
    ("f32", 1, 1, 1, 32, 1, 1, 1),
    ("f32", 2, 9, 3, 64, 2, 3, 2),
    ("f32", 1, 6, 2, 68, 2, 2, 3),
    ("f32", 3, 10, 5, 15, 3, 5, 4),
    ("f32", 1, 14, 35, 132, 3, 7, 2),
    ("bf16", 2, 21, 7, 96, 3, 7, 5),
    ("bf16", 1, 6, 9, 42, 3, 3, 2),
]


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", SHAPES)
def test_convolutions_beside(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9550 + H * W + C, dtype=dtype)
    compare(X, Wqkv, Wo, Wlce, dtype, S, k, heads, "generic")
    compare_backward(X, Wqkv, Wo, Wlce, dtype, heads, S, k, path="generic")


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", [SHAPES[1], SHAPES[3], SHAPES[5],
    ("f32", 132, 30, 14, 64, 2, 2, 1)])      # 1056 workgroups: those that five to a compute unit take in one round
def test_convolution_alone(dtype, B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9560 + H * W + C, dtype=dtype)
    rng = np.random.Generator(np.random.PCG64(9561))
    Ir = np.stack([rng.permutation(S * S)[:k] for _ in range(B * S * S)]).reshape(B, S * S, k).astype(np.int32)
    Y = bra.bra_forward(*(to_device(a, dtype) for a in (X, Wqkv, Wo, Wlce)), S, k, heads, Ir_in=torch.from_numpy(Ir).cuda(), path="generic")
    check_output(to_numpy(Y), run_oracle(X, Wqkv, Wo, Wlce, dict(S=S, k=k, heads=heads), Ir_in=Ir)["Y"], dtype)


@pytest.mark.parametrize("B,C", [(4, 128), (5, 128), (16, 64), (17, 64)])
def test_batches_around_the_small_kernels(B, C):
    # 64 regions per image: the last batch that runs at once and the first that takes the general kernels
    X, Wqkv, Wo, Wlce = make_inputs(B, 32, 32, C, seed=9570 + C, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", 8, 2, C // 32, "generic", images=[0, B - 1])
    Xd, Wd, Wod, Wld = (to_device(a, "f32") for a in (X, Wqkv, Wo, Wlce))
    Y, Ir = bra.bra_forward(Xd, Wd, Wod, Wld, 8, 2, C // 32, want_Ir=True, path="generic")
    assert torch.equal(Ir, bra.bra_route(Xd, Wd, 8, 2, C // 32))


@pytest.mark.parametrize("dtype,B,H,W,C,heads,S,k", [
    ("f32", 1, 7, 7, 128, 4, 7, 32), ("f32", 1, 7, 7, 128, 4, 7, 33), ("f32", 2, 12, 12, 96, 3, 3, 4),
    ("bf16", 2, 12, 12, 96, 3, 3, 5), ("f32", 1, 9, 21, 80, 4, 3, 3),
])
def test_gradients_around_one_block_of_keys(dtype, B, H, W, C, heads, S, k):
    # 32, 33, 64, 80 and 63 routed keys
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9580 + H * W + k, dtype=dtype)
    compare_backward(X, Wqkv, Wo, Wlce, dtype, heads, S, k, path="generic")
