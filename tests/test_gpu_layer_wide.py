"""Layers in one kernel with 64 output channels per workgroup (16 tiles, binary16, n = 4 and 6) against the separate stage calls, bit for
bit: 16 q + 1 and 16 q + 15 tiles, one to 64 channels in the last group, a last group of which U has only 32."""
import pytest
import torch

from test_gpu_layer import equals_the_stages

pytestmark = pytest.mark.gpu

CASES = [
    # m, r, N, C, K, H, W, as the rule has it on 256 compute units
    (2, 3, 3, 5, 33, 60, 62), (2, 3, 1, 16, 192, 62, 121), (2, 3, 19, 64, 96, 23, 23), (2, 3, 18, 65, 97, 23, 23),
    (4, 3, 10, 16, 256, 34, 34), (4, 3, 7, 20, 130, 57, 41), (4, 3, 16, 96, 128, 39, 39), (4, 3, 1, 64, 64, 220, 228),
    (2, 5, 22, 48, 64, 25, 25), (2, 5, 6, 64, 161, 23, 25),
]


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
def test_64_channels_equal_the_stages(m, r, N, C, K, H, W):
    equals_the_stages(m, r, N, C, K, H, W, torch.float16, True)
