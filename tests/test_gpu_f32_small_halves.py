"""GPU parity of the float32 layer of two launches, whose routed keys are shared out between two wavefronts with 64 channels: a half
without keys, one with a region, both full; halves whose references lie far apart; maps of one region and of a single row of regions;
the largest batch of the two launches and the first of the general kernels."""
import numpy as np
import pytest
import torch

import paper_2303_08810_amd as bra
from parity_util import check_output, run_oracle, to_device, to_numpy
from synthetic_inputs import make_inputs
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("B,S,C", [(1, 7, 64), (2, 3, 64), (1, 8, 128), (3, 2, 128)])
def test_keys_of_the_halves(B, S, C, k):
    X, Wqkv, Wo, Wlce = make_inputs(B, 4 * S, 4 * S, C, seed=9890 + S + C, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", S, k, C // 32, "generic")


def test_one_region():
    X, Wqkv, Wo, Wlce = make_inputs(2, 4, 4, 64, seed=9891, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", 1, 1, 2, "generic")


@pytest.mark.parametrize("C", [64, 128])
@pytest.mark.parametrize("lift", [-60.0, 30.0, 60.0])
def test_references_far_apart(C, lift):
    """Scores of the last two routed regions are `lift` above those of the first two (natural units).  A score of 60 is 87 in units of
    log2, where float32 is spaced 7.6e-6: the 31 additions of its product leave about 2e-5 of random error, 1.5e-5 of every weight, and
    1e-4 is above that for outputs of size 4; a lift of 200, spaced four times as wide, exceeded the bar by half."""
    S, k, heads = 3, 4, C // 32
    X, Wqkv, Wo, Wlce = make_inputs(1, 12, 12, C, seed=9892, dtype="f32")
    X[..., 0] = 1.0
    X[:, :, :, 1] = 0.0
    X[:, 4:, :, 1] = 1.0             # regions 3 to 8
    Wqkv[:2, :] = 0.0
    Wqkv[0, 0:C:32] = 1.0
    Wqkv[1, C:2 * C:32] = np.float32(lift * np.sqrt(32.0))
    Ir = np.broadcast_to(np.array([0, 1, 5, 8], np.int32), (1, 9, k)).copy()
    Y = bra.bra_forward(*(to_device(a, "f32") for a in (X, Wqkv, Wo, Wlce)), S, k, heads, Ir_in=torch.from_numpy(Ir).cuda(), path="generic")
    check_output(to_numpy(Y), run_oracle(X, Wqkv, Wo, Wlce, dict(S=S, k=k, heads=heads), Ir_in=Ir)["Y"], "f32")


@pytest.mark.parametrize("B", [21, 22])
def test_largest_batch(B):
    X, Wqkv, Wo, Wlce = make_inputs(B, 32, 32, 64, seed=9893, dtype="f32")
    compare(X, Wqkv, Wo, Wlce, "f32", 8, 3, 2, "generic", images=[0, B - 1])
