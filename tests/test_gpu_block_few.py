"""GPU parity of the block's MLP half where 16 tokens to a workgroup share the hidden units among its wavefronts: fewer and more units than wavefronts have
steps for, remainders of them, tokens that 16 does not divide, a single one, both sides of the line; and of the LayerNorm kernels of few tokens."""
import pytest

from test_gpu_block import compare_block, inputs

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, W, C, heads, S, k, hidden)
    (1, 1, 1, 128, 4, 1, 1, 64),         # one token, two wavefronts with units
    (1, 5, 7, 128, 4, 1, 1, 128),
    (2, 7, 7, 128, 4, 7, 3, 384),        # two and one blocks of units
    (1, 9, 5, 192, 6, 1, 1, 64),
    (3, 14, 14, 192, 6, 7, 5, 576),      # three and two
    (1, 6, 9, 192, 3, 3, 2, 832),
    (1, 14, 14, 256, 8, 7, 4, 768),
    (1, 3, 5, 256, 8, 1, 1, 320),
    (16, 16, 16, 256, 8, 4, 2, 256),     # 4096 tokens
    (1, 17, 241, 192, 6, 1, 1, 192),     # 4097: the other kernel
    (1, 64, 66, 128, 4, 2, 1, 192),      # 4224: the other kernel, 4 wavefronts
    (1, 14, 14, 768, 24, 7, 4, 768),     # several chunks of channels per lane
    (1, 28, 28, 320, 10, 7, 4, 320),
    (1, 35, 28, 320, 10, 7, 4, 320),     # beyond that line
]


@pytest.mark.parametrize("B,H,W,C,heads,S,k,hidden", SHAPES)
def test_few_tokens(B, H, W, C, heads, S, k, hidden):
    X, P = inputs(B, H, W, C, seed=9960 + H * W + C, hidden=hidden)
    compare_block(X, P, S, k, heads, images=sorted({0, B - 1}))


def test_few_tokens_in_place():
    X, P = inputs(2, 14, 14, 192, seed=9961)
    compare_block(X, P, 7, 4, 6, in_place=True)
