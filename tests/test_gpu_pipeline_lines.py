"""GPU parity on both sides of the lines between the kernels specialised by channel count and the general pipeline, for
regions of 2 to 64 tokens: the layer against the oracle with the index of bra_route, and with that index given, which some of 16 and 64 tokens
per region send to the other pipeline, within the scratch that is asked for."""
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import check_output, run_oracle, to_device, to_numpy
from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu

LINES = [  # (B, H, W, C, S, k)
    (32, 14, 7, 256, 7, 4),                                  # 2 tokens
    (42, 14, 14, 256, 7, 3), (84, 14, 14, 128, 7, 3),        # 4
    (66, 14, 14, 256, 7, 3), (67, 14, 14, 256, 7, 3),        # what the general pipeline needs fits the built-in scratch, and not
    (133, 14, 14, 128, 7, 3), (134, 14, 14, 128, 7, 3),
    (36, 14, 28, 256, 7, 2), (39, 14, 28, 256, 7, 2),        # 8
    (18, 28, 28, 256, 7, 2), (20, 28, 28, 256, 7, 2),        # 16
    (2, 28, 28, 128, 7, 3), (10, 28, 28, 128, 7, 4), (11, 28, 28, 128, 7, 4),
    (20, 28, 28, 128, 7, 8), (21, 28, 28, 128, 7, 8),
    (11, 28, 28, 64, 7, 4), (12, 28, 28, 64, 7, 4), (26, 28, 28, 64, 7, 4), (27, 28, 28, 64, 7, 4),
    (9, 56, 56, 128, 7, 1), (10, 56, 56, 128, 7, 1),         # 64
    (10, 56, 56, 128, 7, 2), (11, 56, 56, 128, 7, 2),
    (5, 56, 56, 64, 7, 3), (6, 56, 56, 64, 7, 3),            # with a given index
    (10, 56, 56, 64, 7, 2), (11, 56, 56, 64, 7, 2),
    (2, 56, 112, 64, 7, 2),                                  # 128
    (21, 128, 128, 64, 16, 1), (22, 128, 128, 64, 16, 1),    # 256 regions of 64
    (84, 64, 64, 64, 16, 1), (85, 64, 64, 64, 16, 1),        # and of 16
    (27, 64, 64, 256, 16, 1), (28, 64, 64, 256, 16, 1),
]


@pytest.mark.parametrize("B,H,W,C,S,k", LINES)
def test_lines(B, H, W, C, S, k):
    arrays = make_inputs(B, H, W, C, seed=7900 + B + C, dtype="bf16")
    some = [0, B - 1]
    compare(*arrays, "bf16", S, k, C // 32, "mfma", images=some)
    X, Wqkv, Wo, Wlce = (to_device(a, "bf16") for a in arrays)
    need = bra.workspace_bytes(bra.make_shape(B, H, W, C, C // 32, S, k, torch.bfloat16))
    buffer = torch.full((need + 4096,), 77, dtype=torch.uint8, device=X.device)
    Ir = bra.bra_route(X, Wqkv, S, k, C // 32)
    Y = bra.bra_forward(X, Wqkv, Wo, Wlce, S, k, C // 32, Ir_in=Ir, ws=buffer[:need])
    torch.cuda.synchronize()
    assert bool((buffer[need:] == 77).all())
    Ir = Ir.cpu().numpy()[some]
    ref = run_oracle(arrays[0][some], *arrays[1:], dict(S=S, k=k, heads=C // 32), Ir_in=Ir)
    check_output(to_numpy(Y)[some], ref["Y"], "bf16")
