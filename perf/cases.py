"""Timing cases of the framework: what its users run, through the public entry points.

A case is one call: the forward pass of a BRA layer ("forward"; "padded" for maps whose sides S
does not divide), one whole block around it ("block"), or the gradients of the layer
("backward").  Shapes are the stage shapes of synthetic_inputs.py (224^2 classification, 512^2
dense prediction, the ViT adaptation, S = 16 on a detection-sized map), at a serving batch of one
image and at training batches, in bf16 and in float32.

Inputs are feature maps with spatial structure: white noise plus an offset per region (the
`smooth` recipe of synthetic_inputs.py), weights scaled as there.
"""
from __future__ import annotations

import math

import torch

import paper_2303_08810_amd as bra

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
EXPANSION = 3   # hidden = 3 C in the block's MLP


def case(name, op, dtype, B, H, W, C, heads, S, k, want_Ir=False):
    return dict(name=name, op=op, dtype=dtype, B=B, H=H, W=W, C=C, heads=heads, S=S, k=k, want_Ir=want_Ir)


def listed():
    return [
        # one image through a second-stage-sized layer in float32: launches and latency
        case("fwd_single_f32", "forward", "f32", 1, 28, 28, 64, 2, 7, 4),
        # one 224^2 image at the first stage, served in bf16
        case("fwd_single_stage1", "forward", "bf16", 1, 56, 56, 64, 2, 7, 1),
        # a classification batch at the first stage, the routing kept for the backward pass
        case("fwd_stage1_b64", "forward", "bf16", 64, 56, 56, 64, 2, 7, 1, True),
        # a classification batch at the third stage (regions of 2 x 2 tokens)
        case("fwd_stage3_b64", "forward", "bf16", 64, 14, 14, 256, 8, 7, 16),
        # dense prediction on 512^2 inputs, first stage (regions of 256 tokens)
        case("fwd_dense512_b2", "forward", "bf16", 2, 128, 128, 64, 2, 8, 4),
        # detection-sized first-stage map whose sides S = 16 does not divide
        case("fwd_padded_s16_b2", "padded", "bf16", 2, 200, 300, 64, 2, 16, 4),
        # the plain-ViT adaptation: heads of 64 channels, C = 768
        case("fwd_vit_b8", "forward", "bf16", 8, 32, 32, 768, 12, 8, 12),
        # float32 inference of the first stage
        case("fwd_stage1_f32_b16", "forward", "f32", 16, 56, 56, 64, 2, 7, 1),
        # one whole block at the second stage
        case("block_stage2_b64", "block", "bf16", 64, 28, 28, 128, 4, 7, 4),
        # training: gradients at the first stage, at the wide variant's third stage, and in float32
        case("bwd_stage1_b64", "backward", "bf16", 64, 56, 56, 64, 2, 7, 1),
        case("bwd_wide_stage3_b64", "backward", "bf16", 64, 14, 14, 384, 12, 7, 16),
        case("bwd_stage2_f32_b8", "backward", "f32", 8, 28, 28, 128, 4, 7, 4),
    ]


# channels -> (head counts, largest region side): maps get smaller as channels grow
CHANNELS = {64: ((2,), 16), 96: ((3,), 14), 128: ((4,), 12), 192: ((6,), 8), 256: ((8,), 6),
            384: ((12,), 4), 512: ((16,), 4), 768: ((12, 24), 4)}
F32_ELEMENTS = 16 * 56 * 56 * 64   # the largest float32 tensor among the listed cases


def _weight(c):
    """Rough cost of a case in byte equivalents at bf16 matrix rates."""
    w = work(c)
    return max(w["bytes"], w["flops"] / 300)


def draw(rng):
    log = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999))))
    most = {"forward": 0, "padded": 0, "block": 0, "backward": 0}
    for c in listed():
        if c["dtype"] == "bf16":
            most[c["op"]] = max(most[c["op"]], _weight(c))
    f32_most = {c["op"]: work(c)["flops"] for c in listed() if c["dtype"] == "f32"}
    f32_most["padded"] = f32_most["block"] = f32_most["forward"]
    while True:
        op = rng.choice(["forward"] * 9 + ["padded"] * 2 + ["block"] * 4 + ["backward"] * 5)
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        C = rng.choice(list(CHANNELS))
        heads, side = rng.choice(CHANNELS[C][0]), CHANNELS[C][1]
        S = rng.choice([7, 7, 7, 8, 16] if C <= 128 else [7, 7, 8])
        rh = log(1 if C >= 256 else 2, side)
        rw = rh if rng.random() < 0.6 else log(1 if C >= 256 else 2, side)
        H, W = S * rh, S * rw
        k = log(1, min(S * S, 49, max(1, 1024 // (rh * rw))))
        B = log(1, 64)
        if op == "padded":
            if rh < 2 or rw < 2:
                continue
            H, W = H - rng.randrange(0, min(S, H)), W - rng.randrange(1, min(S, W))
            if -(-H // S) != rh or -(-W // S) != rw:
                continue
        c = dict(op=op, dtype=dtype, B=B, H=H, W=W, C=C, heads=heads, S=S, k=k,
                 want_Ir=op == "forward" and rng.random() < 0.5)
        while c["B"] > 1 and _too_large(c, most, f32_most):
            c["B"] -= 1
        if not _too_large(c, most, f32_most):
            return c


def _too_large(c, most, f32_most):
    if c["dtype"] == "f32" and (c["B"] * c["H"] * c["W"] * c["C"] > F32_ELEMENTS or work(c)["flops"] > f32_most[c["op"]]):
        return True
    return _weight(c) > most[c["op"]]


def _randn(gen, *shape, scale=1.0):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32) * scale


def prepare(case, seed):
    c = case
    B, H, W, C, S, dt = c["B"], c["H"], c["W"], c["C"], c["S"], DTYPES[c["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(20230308 + seed)
    offset = _randn(gen, B, S, S, C)
    rh, rw = -(-H // S), -(-W // S)
    X = _randn(gen, B, H, W, C) + offset.repeat_interleave(rh, 1)[:, :H].repeat_interleave(rw, 2)[:, :, :W]
    s = {"case": c, "X": X.to(dt), "Wqkv": _randn(gen, C, 3 * C, scale=C ** -0.5).to(dt),
         "Wo": _randn(gen, C, C, scale=C ** -0.5).to(dt), "Wlce": _randn(gen, C, 5, 5, scale=0.2).to(dt)}
    if c["op"] == "forward":
        # a program that calls one layer again and again keeps its workspace
        s["ws"] = bra.alloc_workspace(bra.make_shape(B, H, W, C, c["heads"], S, c["k"], dt), s["X"].device)
    elif c["op"] == "backward":
        s["Ir"] = bra.bra_route(s["X"], s["Wqkv"], S, c["k"], c["heads"])
        s["dY"] = _randn(gen, B, H, W, C, scale=0.01).to(dt)
    elif c["op"] == "block":
        hidden = EXPANSION * C
        s["params"] = dict(
            Wpos=_randn(gen, C, 3, 3, scale=1 / 3).to(dt), bpos=_randn(gen, C, scale=0.1),
            ln1_g=1 + _randn(gen, C, scale=0.1), ln1_b=_randn(gen, C, scale=0.1),
            Wqkv=s["Wqkv"], Wo=s["Wo"], Wlce=s["Wlce"],
            ln2_g=1 + _randn(gen, C, scale=0.1), ln2_b=_randn(gen, C, scale=0.1),
            W1=_randn(gen, C, hidden, scale=C ** -0.5).to(dt), b1=_randn(gen, hidden, scale=0.1),
            W2=_randn(gen, hidden, C, scale=hidden ** -0.5).to(dt), b2=_randn(gen, C, scale=0.1))
    return s


def run(state):
    s, c = state, state["case"]
    if c["op"] == "forward":
        return bra.bra_forward(s["X"], s["Wqkv"], s["Wo"], s["Wlce"], c["S"], c["k"], c["heads"],
                               want_Ir=c["want_Ir"], ws=s["ws"])
    if c["op"] == "padded":
        return bra.bra_forward_padded(s["X"], s["Wqkv"], s["Wo"], s["Wlce"], c["S"], c["k"], c["heads"])
    if c["op"] == "block":
        return bra.bra_block_forward(s["X"], s["params"], c["S"], c["k"], c["heads"])
    return bra.bra_backward(s["X"], s["Wqkv"], s["Wo"], s["Wlce"], s["Ir"], s["dY"], c["S"], c["heads"])


def work(case):
    """Bytes: every input read once, every output written once.  Flops: 2 per multiply-add."""
    c = case
    N, C, R, k = c["H"] * c["W"], c["C"], c["S"] ** 2, c["k"]
    eb = 2 if c["dtype"] == "bf16" else 4
    kn = k * -(-c["H"] // c["S"]) * -(-c["W"] // c["S"])
    weights = (4 * C * C + 25 * C) * eb
    routing = N * C + 4 * R * C * C + 2 * R * R * C
    forward = 8 * N * C * C + routing + 4 * N * kn * C + 50 * N * C
    index = 4 * c["B"] * R * k
    if c["op"] == "backward":
        # Q, K, V and O again (nothing but X is kept), dO, dWo, dX, dWqkv; S, O, dP, dV, dQ, dK; three 5 x 5 passes
        flops = c["B"] * (22 * N * C * C + 12 * N * kn * C + 150 * N * C)
        return {"bytes": 3 * c["B"] * N * C * eb + weights + 4 * (4 * C * C + 25 * C) + index, "flops": flops}
    data = 2 * c["B"] * N * C * eb
    if c["op"] == "block":
        hidden = EXPANSION * C
        return {"bytes": data + weights + (9 * C + 2 * C * hidden) * eb + 4 * (6 * C + hidden),
                "flops": c["B"] * (forward + 4 * N * C * hidden + 18 * N * C)}
    return {"bytes": data + weights + (index if c["want_Ir"] else 0), "flops": c["B"] * forward}


def tolerance(case):
    # bf16: independent roundings of the intermediate tensors; indices may differ at near ties
    return {"rel": 1e-2, "differ": 1e-3} if case["dtype"] == "bf16" else {"rel": 1e-5, "differ": 1e-3}
