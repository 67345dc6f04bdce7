"""Values that are not finite come out where the formulas put them: nowhere dropped, nowhere spread."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import to_device
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
