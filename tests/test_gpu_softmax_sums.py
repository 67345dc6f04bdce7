"""The softmax denominators and the row statistics of the backward are sums of float32 weights, also where the weights
enter their product as bf16: one key of weight 1 and 769 of weight 1 / 255, which bf16 rounds up by 0.4 %.  In exact
arithmetic the probabilities are 255 / 1024 and 1 / 1024, and every stored number that is checked here is a bf16 number."""
import math

import pytest
import torch

import paper_2303_08810_amd as bra

pytestmark = pytest.mark.gpu

KEYS = 770


def layer(B, rh, rw, S, C, heads, values, keys=KEYS):
    """X, Wqkv, Wo, Wlce, routing: all queries attend the tokens of the first k regions, Q K^T is 0 for the image's first
    token and -log2(255) for the others (with scale ln 2 the exponent of 2), V is 1 on the first token or on the others."""
    H, W, k, d = S * rh, S * rw, keys // (rh * rw), C // heads
    assert k * rh * rw == keys and k <= S * S
    X = torch.zeros(B, H, W, C, device="cuda")
    X[..., 0] = 1.0
    X[:, 0, 0, 0] = 0.0
    X[..., 1] = 1.0
    X[:, 0, 0, 2] = 1.0
    Wqkv = torch.zeros(C, 3 * C, device="cuda")
    Wqkv[1, 0:C:d] = Wqkv[1, 1:C:d] = 1.0
    Wqkv[0, C:2 * C:d] = -8.0
    Wqkv[0, C + 1:2 * C:d] = 8.0 - math.log2(255.0)          # its bf16 rounding is off by 1e-6
    Wqkv[2 if values == "first" else 0, 2 * C:] = 1.0
    bf = [t.bfloat16() for t in (X, Wqkv, torch.eye(C, device="cuda"), torch.zeros(C, 5, 5, device="cuda"))]
    Ir = torch.arange(k, dtype=torch.int32, device="cuda").expand(B, S * S, k).contiguous()
    return bf, Ir, k


# (B, rh, rw, S, C, heads): 16, 32, 64 and 128 queries at a time
@pytest.mark.parametrize("B,rh,rw,S,C,heads", [(1, 2, 7, 8, 192, 6), (2, 2, 11, 7, 192, 3), (1, 7, 11, 4, 192, 6),
                                               (19, 10, 11, 3, 192, 3), (19, 10, 11, 3, 192, 6)])
def test_forward_denominators(B, rh, rw, S, C, heads):
    (X, Wqkv, Wo, Wlce), Ir, k = layer(B, rh, rw, S, C, heads, "first")
    Y = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, heads, Ir_in=Ir, scale=math.log(2.0), path="mfma")
    assert torch.equal(Y.float(), torch.full_like(Y.float(), 255 / 1024))


# More than 64 regions of 64 tokens: by 64 queries on 5.1 x 2^20 values (also C = 128 where less scratch is asked for), and in the
# general pipeline on fewer.  255 / 2302 is 226.86 units of the last place, with weights rounded to bf16 226.08
@pytest.mark.parametrize("B,C,heads", [(16, 64, 2), (1, 64, 2), (7, 128, 4)])
def test_forward_denominators_of_many_regions(B, C, heads):
    (X, Wqkv, Wo, Wlce), Ir, k = layer(B, 8, 8, 9, C, heads, "first", keys=2048)
    want = torch.tensor(255 / 2302).bfloat16().float().item()
    Y = bra.bra_forward(X, Wqkv, Wo, Wlce, 9, k, heads, Ir_in=Ir, scale=math.log(2.0), path="mfma")
    assert torch.equal(Y.float(), torch.full_like(Y.float(), want))
    if bra.workspace_bytes(bra.make_shape(B, 72, 72, C, heads, 9, k, torch.bfloat16)) > bra.STATIC_SCRATCH_BYTES and C == 128:
        Y = torch.empty_like(X)
        bra.bra_forward_static(X, Wqkv, Wo, Wlce, 9, k, heads, out=Y, Ir_in=Ir, scale=math.log(2.0))
        assert torch.equal(Y.float(), torch.full_like(Y.float(), want))


# Few regions and few keys: 288 pairs of image and head, 96 keys, fewer blocks of keys than the image-resident attention takes.  With
# V = 161 / 128, 234.6 units of the last place, with weights rounded to bf16 234.35
def test_forward_denominators_of_few_regions():
    (X, Wqkv, Wo, Wlce), Ir, k = layer(12, 2, 2, 5, 768, 24, "first", keys=96)
    Wqkv[2, 2 * 768:] = 161 / 128
    Y = bra.bra_forward(X, Wqkv, Wo, Wlce, 5, k, 24, Ir_in=Ir, scale=math.log(2.0), path="mfma")
    want = torch.tensor(161 / 128 * 255 / 350).bfloat16().float().item()
    assert torch.equal(Y.float(), torch.full_like(Y.float(), want))


# a wavefront per region (16 and 32 tokens), four wavefronts per tile, 64 and 128 tokens per workgroup
BACKWARD = [(6, 2, 7, 8, 64, 1), (6, 2, 11, 7, 64, 2), (1, 2, 7, 8, 64, 2), (1, 2, 11, 7, 64, 1), (3, 7, 11, 4, 64, 2),
            (57, 10, 11, 3, 64, 1), (57, 10, 11, 3, 64, 2)]


def gradients(B, rh, rw, S, C, heads, values):
    (X, Wqkv, Wo, Wlce), Ir, k = layer(B, rh, rw, S, C, heads, values)
    dY = torch.zeros_like(X)
    dY.view(B, -1, C)[:, :512] = 1.0
    dWqkv = bra.bra_backward(X, Wqkv, Wo, Wlce, Ir, dY, S, heads, scale=math.log(2.0), path="mfma")[1]
    return dWqkv.view(C, 3, C)


@pytest.mark.parametrize("B,rh,rw,S,C,heads", BACKWARD)
def test_backward_denominators(B, rh, rw, S, C, heads):
    # dV = P^T dO over 512 queries: 512 / 1024 for each of 769 keys, 512 * 255 / 1024 for the first
    dW = gradients(B, rh, rw, S, C, heads, "first")
    assert torch.allclose(dW[0, 2], torch.full((C,), B * 769 * 0.5, device="cuda"), rtol=1e-5)
    assert torch.allclose(dW[2, 2], torch.full((C,), B * 127.5, device="cuda"), rtol=1e-5)


@pytest.mark.parametrize("B,rh,rw,S,C,heads", BACKWARD)
def test_backward_row_sums(B, rh, rw, S, C, heads):
    # V is 1 on the others: with d channels per head D = d 769 / 1024, dS = d 255 / 1024 / 1024 for each of them and, K being
    # -8 there in channel 0 of a head, dQ = ln 2 * 769 dS * -8 at each of the 512 queries.  dS is a bf16 number; the bound
    # is one rounding to bf16 of dQ, 2^-9, and the float32 sums
    dW = gradients(B, rh, rw, S, C, heads, "others")
    d = C // heads
    dQ = -8.0 * math.log(2.0) * 769 * d * 255 / 1024 / 1024
    assert torch.allclose(dW[1, 0, ::d], torch.full((heads,), B * 512 * dQ, device="cuda"), rtol=2.1e-3)


# The reference of the exponentials has to move from block to block: every 16 keys the scores go up by `step` powers of two
# (beyond the range of float32 for 200), down again, or up and down.  All weights are powers of two, so nothing but the
# result is rounded.
def steps(B, rh, rw, S, k, C, heads, step, order):
    n, R = rh * rw, S * S
    g = torch.Generator(device="cuda").manual_seed(9990 + n)
    T = torch.randint(-3, 4, (B, R, n, C), generator=g, device="cuda").float()      # tokens by region
    T[..., 0], T[..., 1] = 0.0, 1.0
    group = torch.arange(k * n, device="cuda") // 16
    top = int(group[-1])
    rank = {"up": group, "down": top - group, "zigzag": torch.where(group % 2 == 0, group, top - group)}[order]
    T[:, :k, :, 0] = rank.view(k, n).float()
    X = T.view(B, S, S, rh, rw, C).permute(0, 1, 3, 2, 4, 5).reshape(B, S * rh, S * rw, C).contiguous()
    d = C // heads
    Wqkv = torch.zeros(C, 3 * C, device="cuda")
    Wqkv[1, 0:C:d] = 1.0
    Wqkv[0, C:2 * C:d] = step
    channel = torch.arange(C, device="cuda")
    Wqkv[2 + channel % (C - 2), 2 * C + channel] = 1.0
    Ir = torch.arange(k, dtype=torch.int32, device="cuda").expand(B, R, k).contiguous()
    args = [t.bfloat16() for t in (X, Wqkv, torch.eye(C, device="cuda"), torch.zeros(C, 5, 5, device="cuda"))]
    V = T[:, :k].reshape(B, k * n, C)[..., 2 + channel % (C - 2)].double()
    P = torch.exp2((rank - rank.max()).double() * step)
    return args, Ir, V, P / P.sum()


@pytest.mark.parametrize("order", ["up", "down", "zigzag"])
@pytest.mark.parametrize("step", [4, 10, 200])
@pytest.mark.parametrize("B,rh,rw,S,k,C,heads", [(1, 2, 7, 7, 20, 192, 6), (2, 5, 5, 5, 11, 192, 3), (1, 8, 8, 4, 7, 192, 3),
                                                 (19, 10, 11, 3, 7, 192, 6)])
def test_moving_reference(B, rh, rw, S, k, C, heads, step, order):
    (X, Wqkv, Wo, Wlce), Ir, V, P = steps(B, rh, rw, S, k, C, heads, step, order)
    Y = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, heads, Ir_in=Ir, scale=math.log(2.0), path="mfma")
    ref = (P[None, :, None] * V).sum(1)
    err = (Y.double().view(B, -1, C) - ref[:, None]).abs() / (ref[:, None].abs() + 2.0 ** -12)
    assert float(err.max()) <= 2.0 ** -8


@pytest.mark.parametrize("order", ["up", "zigzag"])
@pytest.mark.parametrize("step", [4, 10, 200])
@pytest.mark.parametrize("B,rh,rw,S,C,heads", [(6, 2, 7, 7, 64, 2), (6, 5, 5, 5, 64, 1), (1, 5, 5, 5, 64, 2), (3, 8, 8, 4, 128, 4),
                                               (57, 10, 11, 3, 64, 2)])
def test_moving_reference_backward(B, rh, rw, S, C, heads, step, order):
    k = min(7, S * S)
    (X, Wqkv, Wo, Wlce), Ir, V, P = steps(B, rh, rw, S, k, C, heads, step, order)
    dY = torch.randint(-2, 3, X.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9991)).bfloat16()
    dW = bra.bra_backward(X, Wqkv, Wo, Wlce, Ir, dY, S, heads, scale=math.log(2.0), path="mfma")[1].double()
    # every query has the same probabilities: dV = P^T dO; dS = P (dP - sum P dP), dK is its sum in channel 0 of each head
    d, n = C // heads, rh * rw
    g = dY.double().view(B, -1, heads, d).sum(1)                                    # dO summed over the queries
    dP = torch.einsum("bhd,bkhd->bkh", g, V.view(B, -1, heads, d))
    dS = P[None, :, None] * (dP - torch.einsum("k,bkh->bh", P, dP)[:, None])
    keys = X.view(B, S, rh, S, rw, C).permute(0, 1, 3, 2, 4, 5).reshape(B, S * S, n, C)[:, :k].reshape(B, k * n, C).double()
    want_k = math.log(2.0) * torch.einsum("bkc,bkh->ch", keys, dS)
    want_v = torch.einsum("bkc,k,bhd->chd", keys, P, g).reshape(C, C)
    # Rows 0 and 1 (the group's number, up to 48, and the constant) are left out for dK: sum_t dK[t] is 0 and only the
    # roundings of dK, times the number, are left of it.  Else as in test_gpu_backward.py, 1e-2 of the largest element of a
    # block: an element is a sum over the keys of products that carry four bf16 roundings
    want_k, got_k, got_v = want_k[2:], dW[2:, C:2 * C:d], dW[:, 2 * C:]
    assert float((got_v - want_v).abs().max()) <= 1e-2 * float(want_v.abs().max())
    assert float((got_k - want_k).abs().max()) <= 1e-2 * float(want_k.abs().max())
