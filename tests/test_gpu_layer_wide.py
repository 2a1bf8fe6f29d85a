"""Layers in one kernel with 64 output channels per workgroup (binary32: 32; 16 tiles, n = 4 and 6) against the separate stage calls, bit
for bit: 16 q + 1 and 16 q + 15 tiles, one channel to all in the last group, a last group of which U has only 32."""
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


CASES_BINARY32 = [
    (2, 3, 3, 24, 128, 110, 110), (2, 3, 3, 64, 33, 46, 94), (4, 3, 22, 16, 96, 25, 25), (4, 3, 9, 5, 17, 60, 61), (4, 3, 15, 40, 65, 29, 26),
    (2, 5, 4, 16, 32, 53, 53),
]


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES_BINARY32)
def test_32_channels_of_binary32_equal_the_stages(m, r, N, C, K, H, W):
    equals_the_stages(m, r, N, C, K, H, W, torch.float32, True)
