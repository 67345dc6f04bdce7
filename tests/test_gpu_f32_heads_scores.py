"""Scores of the float32 gradients where wavefronts share a head of a region: as float64 has them where terms cancel, and without
bounds where a tile of keys has none that counts."""
import numpy as np
import pytest
import torch

import oracle.backward as oracle_backward
import paper_2303_08810_amd as bra
from parity_util import to_device
from synthetic_inputs import make_inputs

pytestmark = pytest.mark.gpu

# 4 x 4 tokens per region and heads of 32 channels: four, two and one wavefronts per head; 25 tokens: two tiles of queries
SHAPES = [  # (B, H, W, C, heads, S, k)
    (2, 16, 16, 128, 4, 4, 4),
    (20, 16, 16, 128, 4, 4, 4),
    (40, 16, 16, 128, 4, 4, 4),
    (2, 20, 20, 128, 4, 4, 4),
    (2, 16, 16, 64, 2, 4, 16),
    (2, 12, 12, 128, 4, 3, 9),
]


def both(X, Wqkv, Wo, Wlce, S, heads, Ir, dY):
    got = bra.bra_backward(*(to_device(a, "f32") for a in (X, Wqkv, Wo, Wlce)), torch.from_numpy(Ir).cuda(), to_device(dY, "f32"), S, heads)
    ref = oracle_backward.bra_backward(X, Wqkv, Wo, Wlce, dY, Ir, S=S, heads=heads)
    return [(name, g.cpu().numpy().astype(np.float64).reshape(ref[name].shape), ref[name]) for name, g in zip(("dX", "dWqkv", "dWo", "dWlce"), got)]


def check(name, got, ref, bar=1e-5):
    error = float(np.abs(got - ref).max() / np.abs(ref).max()) if np.isfinite(got).all() else np.inf
    assert error <= bar, (name, error)


def routing(B, S, k, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return np.stack([np.stack([rng.permutation(S * S)[:k] for _ in range(S * S)]) for _ in range(B)]).astype(np.int32)


# Three channels of every head whose terms, up to 2^20, cancel: 1000 t - 999 t - t with a t of each key's own.  All of Q and K is whole numbers,
# partial sums lie below 2^24, and so the float32 scores are exact; scaled before they are multiplied, terms leave up to 2^20 2^-24 = 6 % of a weight
# (5e-3 of the largest value of dX).  What is left is the error of any float32 pass (measured below 1e-6).
@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
def test_cancelling_terms(B, H, W, C, heads, S, k):
    _, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9970 + H + C + k, dtype="f32")
    rng = np.random.Generator(np.random.PCG64(9971))
    X = rng.integers(-1, 2, (B, H, W, C)).astype(np.float32)
    dY = rng.standard_normal(X.shape).astype(np.float32)
    Wqkv[:, :2 * C] = 0
    for c in range(2 * C):               # Q and K are sums of four channels
        Wqkv[2 + rng.permutation(C - 2)[:4], c] = rng.choice([-1, 1], 4)
    X[..., 0] = 1
    X[..., 1] = rng.integers(-1000, 1001, X.shape[:3])
    d = C // heads
    for h in range(heads):
        for u, q in enumerate((1000, -999, -1)):
            Wqkv[:, h * d + u] = 0
            Wqkv[0, h * d + u] = q
            Wqkv[:, C + h * d + u] = 0
            Wqkv[1, C + h * d + u] = 1
    Wqkv[1, 2 * C:] = 0                  # t enters K in those channels, and nothing else
    for name, got, ref in both(X, Wqkv, Wo, Wlce, S, heads, routing(B, S, k, 9972), dY):
        # the gradients of the three channels are a thousand times the others': without their columns and rows
        if name == "dWqkv":
            keep = np.array([c % d > 2 for c in range(C)])
            for part in range(3):
                cols = slice(part * C, (part + 1) * C)
                check((name, part), got[2:, cols][:, keep], ref[2:, cols][:, keep])
        elif name == "dX":
            check(name, got[..., 2:], ref[..., 2:])
        else:
            check(name, got, ref)


# One query whose scores overflow to -inf with all keys of one routed region: their weights are zero, as in float64 (exp(-1e39)), wherever the
# region stands among the routed ones
@pytest.mark.parametrize("B,H,W,C,heads,S,k", SHAPES)
@pytest.mark.parametrize("place", [0, 1, -1])
def test_tile_without_weights(B, H, W, C, heads, S, k, place):
    X, Wqkv, Wo, Wlce = make_inputs(B, H, W, C, seed=9980 + H + C + k, dtype="f32")
    rng = np.random.Generator(np.random.PCG64(9981))
    dY = rng.standard_normal(X.shape).astype(np.float32)
    Ir = routing(B, S, k, 9982)
    rh, rw = H // S, W // S
    region = int(Ir[0, 0, place])        # routed from region 0, whose first token is the query
    X[..., 0] = X[..., 1] = 0
    X[0, rh * (region // S):rh * (region // S) + rh, rw * (region % S):rw * (region % S) + rw, 1] = 1
    X[0, 0, 0, 0] = 1
    Wqkv[0], Wqkv[1] = 0, 0
    Wqkv[:, 5] = Wqkv[:, C + 5] = 0
    Wqkv[0, 5] = 1e20                    # Q of the query
    Wqkv[1, C + 5] = -1e20               # K of the region
    for name, got, ref in both(X, Wqkv, Wo, Wlce, S, heads, Ir, dY):
        if name == "dX":                 # the two channels overflow in float32
            got, ref = got[..., 2:], ref[..., 2:]
        elif name == "dWqkv":            # and these columns are 1e20 times the others
            got, ref = np.delete(got, [5, C + 5], axis=1), np.delete(ref, [5, C + 5], axis=1)
        check(name, got, ref)
