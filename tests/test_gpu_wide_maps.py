"""Maps whose rows are so long that a few of them span 2 GiB: the depth-wise kernels take shorter strips, and beyond that
the kernels with 64-bit addresses.  Checked at sampled tokens against the formulas in float64, from the GPU's routing."""
import pytest
import torch

import paper_2303_08810_amd as bra

pytestmark = pytest.mark.gpu


def layer(H, W, C, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *shape, scale=1.0: (torch.randn(*shape, generator=g, device="cuda", dtype=torch.bfloat16) * scale)
    return r(1, H, W, C), r(C, 3 * C, scale=C ** -0.5), r(C, C, scale=C ** -0.5), r(C, 5, 5, scale=0.2)


def window(M, y, x):
    """The 5 x 5 neighbourhood of a token of M [H, W, ...], zero outside."""
    H, W = M.shape[:2]
    out = torch.zeros(5, 5, *M.shape[2:], dtype=torch.float64, device=M.device)
    for dy in range(5):
        for dx in range(5):
            if 0 <= y + dy - 2 < H and 0 <= x + dx - 2 < W:
                out[dy, dx] = M[y + dy - 2, x + dx - 2].double()
    return out


# (H, W, S): strips of 10 rows (the whole map spans 2 GiB), 64-bit addresses (9 rows do); regions of one row each
@pytest.mark.parametrize("H,W,S", [(16, 349536, 16), (9, 621387, 9)])
def test_forward_wide_map(H, W, S):
    C, heads, rw = 192, 6, W // S
    X, Wqkv, Wo, Wlce = layer(H, W, C, seed=9300 + H)
    Y, Ir = bra.bra_forward(X, Wqkv, Wo, Wlce, S, 1, heads, want_Ir=True, path="mfma")
    Wq, Wk, Wv = Wqkv.double().split(C, 1)
    err = ref = 0.0
    for y, x in [(0, 0), (0, W - 1), (H - 1, 0), (H - 1, W - 1), (H // 2, W // 2), (1, 12345), (H - 3, W - 15), (4, rw), (5, rw - 1)]:
        j = int(Ir[0, y * S + x // rw, 0])                        # regions are rows cut into S pieces
        G = X[0, j // S, j % S * rw:(j % S + 1) * rw].double()
        q = (X[0, y, x].double() @ Wq).view(heads, 1, -1)
        k, v = ((G @ w).view(rw, heads, -1).transpose(0, 1).contiguous() for w in (Wk, Wv))
        P = torch.softmax((q * k).sum(-1) * (C // heads) ** -0.5, -1)
        O = (P[..., None] * v).sum(1).view(C) + ((window(X[0], y, x) @ Wv) * Wlce.double().permute(1, 2, 0)).sum((0, 1))
        e = Y[0, y, x].double() - O @ Wo.double()
        err, ref = err + float(e @ e), ref + float((O @ Wo.double()).square().sum())
    assert err ** 0.5 <= 8e-3 * ref ** 0.5, (err / ref) ** 0.5      # the bar of bf16 outputs, see parity_util.check_output


# (H, W, S): the gradient map has three times the pitch
@pytest.mark.parametrize("H,W,S", [(16, 116544, 16), (9, 207135, 9)])
def test_backward_wide_map(H, W, S):
    C, heads, rw, d = 192, 6, W // S, 32
    X, Wqkv, Wo, Wlce = layer(H, W, C, seed=9400 + H)
    dY = X.flip(2) * 0.5
    Ir = torch.arange(S * S, dtype=torch.int32, device="cuda").view(1, -1, 1)       # every region attends itself
    dX, _, _, dWlce = bra.bra_backward(X, Wqkv, Wo, Wlce, Ir, dY, S, heads, path="mfma")
    Wq, Wk, Wv = Wqkv.float().split(C, 1)
    V = (X[0].float().view(-1, C) @ Wv).view(H, W, C)
    dO = (dY[0].float().view(-1, C) @ Wo.float().T).view(H, W, C)
    taps = torch.zeros(C, 5, 5, device="cuda")
    for a in range(5):
        for b in range(5):
            y0, y1, x0, x1 = max(0, 2 - a), min(H, H + 2 - a), max(0, 2 - b), min(W, W + 2 - b)
            taps[:, a, b] = (dO[y0:y1, x0:x1] * V[y0 + a - 2:y1 + a - 2, x0 + b - 2:x1 + b - 2]).sum((0, 1))
    assert float((dWlce - taps).abs().max()) <= 1e-2 * float(taps.abs().max())
    for y, r in [(0, 0), (H - 1, S - 1), (H // 2, 1)]:                              # one region each, all its tokens
        xs = slice(r * rw, (r + 1) * rw)
        x = X[0, y, xs].float()
        D = [torch.zeros(rw, C, device="cuda") for _ in range(3)]
        for h in range(heads):
            c = slice(h * d, (h + 1) * d)
            q, k, v, g = x @ Wq[:, c], x @ Wk[:, c], V[y, xs, c].contiguous(), dO[y, xs, c].contiguous()
            P = torch.softmax(q @ k.T.contiguous() * d ** -0.5, -1)
            dS = g @ v.T.contiguous()
            dS = P * (dS - (P * dS).sum(1, keepdim=True)) * d ** -0.5
            D[0][:, c], D[1][:, c], D[2][:, c] = dS @ k, dS.T.contiguous() @ q, P.T.contiguous() @ g
            del P, dS
        for a in range(5):
            for b in range(5):                                                      # LCE^T
                yy = y - (a - 2)
                if 0 <= yy < H:
                    s = torch.arange(r * rw, (r + 1) * rw, device="cuda") - (b - 2)
                    ok = (s >= 0) & (s < W)
                    D[2] += dO[yy, s.clamp(0, W - 1)] * ok[:, None] * Wlce.float()[:, a, b]
        ref = D[0] @ Wq.T + D[1] @ Wk.T + D[2] @ Wv.T
        err = float((dX[0, y, xs].float() - ref).norm() / ref.norm())
        assert err <= 1e-2, err
