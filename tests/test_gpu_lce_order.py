"""The depth-wise convolution in front of what it is added to, as float32 halves in two maps, and behind it: GPU parity beyond
the lines up to which it runs in front (6 or 9 x 2^20 values in the forward, 14 x 2^20 and more in the gradients; other files hold the sizes
below), and the number of roundings where it does, and where a kernel with the convolution in it takes the shape, at any size.  With taps so large that nothing else shows, Y carries those of V, O and Y
and dX those of dO, dV and dX.  A rounding to bf16 is 1.66e-3 rms of a spread of values: three of them 2.87e-3, four (the
convolution rounded before it is added to) 3.3e-3; the bound lies between."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from oracle import backward as obw
from parity_util import run_oracle, to_device, to_numpy
from synthetic_inputs import make_inputs, round_to_bf16
from test_gpu_backward import compare_backward
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

THREE_ROUNDINGS = 3.1e-3
SHAPES = [  # (B, H, W, C, heads, S, k)
    (1, 28, 28, 192, 6, 7, 2),       # 16 tokens per region
    (1, 30, 35, 128, 2, 5, 2),       # 42
    (2, 16, 64, 192, 3, 2, 1),       # 256
]


def heavy_taps(B, H, W, C, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9900 + H * W + C, dtype="bf16")
    r = np.random.Generator(np.random.PCG64(9901 + C))
    Ir = np.stack([r.permutation(S * S)[:k] for _ in range(B * S * S)]).reshape(B, S * S, k).astype(np.int32)
    return X, Wqkv, Wo, 64 * Wlce, Ir, round_to_bf16(r.standard_normal(X.shape).astype(np.float32))


def rms_error(got, ref):
    return float(np.linalg.norm(to_numpy(got).astype(np.float64).reshape(ref.shape) - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_convolution_rounds_once(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce, Ir, dY = heavy_taps(B, H, W, C, S, k)
    x, wqkv, wo, wlce, dy = (to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce, dY))
    ir = torch.from_numpy(Ir).cuda()
    Y = bra.bra_forward(x, wqkv, wo, wlce, S, k, heads, Ir_in=ir, path="mfma")
    e = rms_error(Y, np.asarray(run_oracle(X, Wqkv, Wo, Wlce, dict(S=S, k=k, heads=heads), Ir_in=Ir)["Y"], np.float64))
    dX = bra.bra_backward(x, wqkv, wo, wlce, ir, dy, S, heads, path="mfma")[0]
    d = rms_error(dX, obw.bra_backward(X, Wqkv, Wo, Wlce, dY, Ir, S=S, heads=heads)["dX"])
    print(f"rms error of Y {e:.3e}, of dX {d:.3e}", flush=True)
    assert e <= THREE_ROUNDINGS and d <= THREE_ROUNDINGS


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (16, 128, 128, 64, 2, 16, 4),    # more than 64 regions, of 64 tokens
    (5, 128, 128, 128, 4, 16, 1),
    (37, 64, 64, 64, 2, 16, 4),      # of 16
    (20, 64, 64, 128, 4, 16, 4),
    (10, 64, 64, 256, 8, 16, 1),
    (64, 14, 28, 384, 12, 7, 4),     # 8 tokens, maps whose convolution the image-resident attention has room for
    (61, 14, 28, 512, 16, 7, 16),
    (64, 10, 20, 768, 24, 5, 8),
])
def test_one_rounding_beyond_the_lines(B, H, W, C, heads, S, k):
    # the other way round: equal scores, so that the attention is a mean of kn values of V and as exact as they are, and a
    # convolution of a third of it, which shows a rounding of the attention before it is added to
    X, Wqkv, Wo, Wlce, Ir, _ = heavy_taps(B, H, W, C, S, k)
    Wqkv[:, :C] = 0
    Wlce = round_to_bf16(Wlce * np.float32(0.3 / 64 / np.sqrt(k * (H // S) * (W // S))))
    x, wqkv, wo, wlce = (to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce))
    Y = bra.bra_forward(x, wqkv, wo, wlce, S, k, heads, Ir_in=torch.from_numpy(Ir).cuda(), path="mfma")
    some = [0, B - 1]      # images are independent of each other
    ref = run_oracle(X[some], Wqkv, Wo, Wlce, dict(S=S, k=k, heads=heads), Ir_in=Ir[some])["Y"]
    e = rms_error(Y[some], np.asarray(ref, np.float64))
    print(f"rms error of Y {e:.3e}", flush=True)
    assert e <= THREE_ROUNDINGS


@pytest.mark.parametrize("B,H,W,C,heads,S,k", [
    (17, 56, 56, 192, 6, 7, 1),      # 9.8 x 2^20 values
    (30, 49, 49, 128, 4, 7, 1),      # 8.8, short rows in the routing
    (62, 14, 28, 512, 16, 7, 16),    # regions of 8 tokens by whole images
    (58, 14, 28, 512, 16, 7, 16),    # and region by region, in front
])
def test_convolution_behind_attention(B, H, W, C, heads, S, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9950, dtype="bf16")
    compare(X, Wqkv, Wo, Wlce, "bf16", S, k, heads, "mfma")


@pytest.mark.parametrize("B,H,W", [(75, 56, 56), (19, 112, 112)])      # 14.4 x 2^20: behind; 14.6, 256 tokens per region: beside
def test_convolution_of_large_gradients(B, H, W):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, 64, seed=9951, dtype="bf16")
    compare_backward(X, Wqkv, Wo, Wlce, "bf16", 2, 7, 1, path="mfma")
