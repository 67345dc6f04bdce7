"""Values that are not finite come out where the formulas put them: nowhere dropped, nowhere spread."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import to_device
from synthetic_inputs import make_inputs
from test_gpu_block import device_params, inputs

pytestmark = pytest.mark.gpu


# (dtype, C, heads, expansion): every place of the GELU: the fused and the streamed MLP kernel, the product's epilogue, float32
@pytest.mark.parametrize("dtype,C,heads,e", [("bf16", 64, 2, 3), ("bf16", 128, 4, 3), ("bf16", 64, 2, 5),
                                             ("bf16", 320, 10, 1), ("f32", 64, 2, 3), ("bf16", 96, 3, 1)])
def test_gelu_keeps_nan(dtype, C, heads, e):
    X, P = inputs(1, 14, 14, C, seed=9900 + C + e, expansion=e, dtype=dtype)
    b1 = P["b1"].copy()
    for value, finite in ((np.nan, False), (np.inf, False), (-np.inf, True)):
        P["b1"] = b1.copy()
        P["b1"][5] = value               # one hidden unit: every output channel of every token takes it
        P["W2"][5] = np.where(P["W2"][5] == 0, 1, P["W2"][5])
        out = bra.bra_block_forward(to_device(X, dtype), device_params(P, dtype), 7, 4, heads).float()
        torch.cuda.synchronize()
        assert bool(torch.isfinite(out).all()) if finite else not bool(torch.isfinite(out).any()), value
        if np.isnan(value):
            assert bool(torch.isnan(out).all())


# O += LCE(V) and dV += LCE^T(dO) on bf16 maps: even and odd widths, one column, several strips
@pytest.mark.parametrize("H,W,C,heads,S", [(14, 14, 64, 2, 7), (21, 7, 128, 2, 7), (40, 1, 64, 1, 1), (24, 50, 192, 6, 2)])
@pytest.mark.parametrize("channel", [2, 5])
def test_depthwise_channels_independent(H, W, C, heads, S, channel):
    X, Wqkv, Wo, Wlce = make_inputs(1, H, W, C, seed=9950 + H + C, dtype="bf16")
    rng = np.random.Generator(np.random.PCG64(9951))
    dY = np.asarray(X) * np.float32(0.5)
    Ir = np.stack([rng.permutation(S * S)[:1] for _ in range(S * S)])[None].astype(np.int32)
    y, x = H // 2, W // 2
    other = np.arange(C) != channel

    def gradients(X, Wqkv, Wo, dY):
        args = [to_device(a, "bf16") for a in (X, Wqkv, Wo, Wlce)]
        out = bra.bra_backward(*args, torch.from_numpy(Ir).cuda(), to_device(dY, "bf16"), S, heads, path="mfma")
        return [g.float().cpu().numpy() for g in out]

    # V overflows in one channel of one token: dWo = O^T dY is finite in every other row
    Xi, Wi = X.copy(), Wqkv.copy()
    Xi[0, y, x, 7] = 2.0 ** 100
    Wi[7] = 0
    Wi[7, 2 * C + channel] = 2.0 ** 40
    dWo = gradients(Xi, Wi, Wo, dY)[2]
    assert np.isfinite(dWo[other]).all() and not np.isfinite(dWo[channel]).any()
    # dO overflows there: dV and its columns of dWqkv = X^T dV are finite in every other channel
    dYi, Woi = dY.copy(), Wo.copy()
    dYi[0, y, x, 9] = 2.0 ** 100
    Woi[:, 9] = 0
    Woi[channel, 9] = 2.0 ** 40
    dW = gradients(X, Wqkv, Woi, dYi)[1][:, 2 * C:]
    assert np.isfinite(dW[:, other]).all() and not np.isfinite(dW[:, channel]).any()


# K^r infinite in one of the last channels, the ones that were repeated where a batch of the routing's steps ran past the end: A^r is
# +-inf in that region's column, by the sign of Q^r there, in bra_route (steps by six) as in bra_forward (by three).  512 channels
# are four steps per slice (eight with more than 64 regions), 320 two and three, 192 one and two; 40 end within a step of 16
@pytest.mark.parametrize("dtype,C,heads,S", [("bf16", 512, 16, 7), ("bf16", 320, 10, 7), ("bf16", 192, 6, 7), ("bf16", 512, 16, 9), ("f32", 512, 16, 7),
                                             ("f32", 40, 1, 7), ("f32", 48, 2, 9), ("f32", 39, 3, 7)])
def test_routing_by_an_infinite_key(dtype, C, heads, S):
    H, region = 2 * S, 5
    X, Wqkv, Wo, Wlce = make_inputs(1, H, H, C, seed=9960 + C + S, dtype=dtype)
    means = X.astype(np.float64).reshape(S, 2, S, 2, C).mean(axis=(1, 3)).reshape(S * S, C)
    Wqkv[7] = 0
    q = (means @ Wqkv.astype(np.float64))[:, C - 2]      # Q^r of the channel (channel 7 of X does not enter)
    assert np.abs(q).min() > 1e-5
    X[..., 7] = 0
    X[0, 2 * (region // S), 2 * (region % S), 7] = 2.0 ** 100
    Wqkv[7, C + C - 2] = 2.0 ** 40
    args = [to_device(a, dtype) for a in (X, Wqkv, Wo, Wlce)]
    Ir = bra.bra_route(*args[:2], S, 3, heads)
    used = bra.bra_forward(*args, S, 3, heads, want_Ir=True)[1]
    assert torch.equal(Ir, used)
    Ir = Ir[0].cpu().numpy()
    assert (Ir[q > 0, 0] == region).all() and (Ir[q < 0] != region).all()
