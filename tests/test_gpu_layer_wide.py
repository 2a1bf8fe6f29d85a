"""Layers in one kernel with 64 output channels per workgroup (binary32: 32; 16 tiles, n = 4 and 6) against the separate stage calls, bit
for bit: 16 q + 1 and 16 q + 15 tiles, one channel to all in the last group, a last group of which U has only 32.  The launched shape is asserted."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova
from test_gpu_layer import equals_the_stages, points_for, workspace

pytestmark = pytest.mark.gpu

CASES = [
    # m, r, N, C, K, H, W, as the rule has it on 256 compute units
    (2, 3, 11, 5, 33, 60, 62), (2, 3, 1, 16, 192, 62, 121), (2, 3, 19, 64, 96, 23, 23), (2, 3, 18, 65, 97, 23, 23),
    (4, 3, 10, 16, 256, 34, 34), (4, 3, 7, 20, 130, 57, 41), (4, 3, 16, 96, 128, 39, 39), (4, 3, 1, 64, 64, 220, 228),
    (2, 5, 22, 48, 64, 25, 25), (2, 5, 6, 64, 161, 23, 25),
]


def is_wide(m, r, N, C, K, H, W, dtype):
    t = nova.nova_make_transforms(points_for(m, r), m, r)
    x, y = torch.zeros((N, C, H, W), dtype=dtype, device="cuda:0"), torch.empty((N, K, H, W), dtype=dtype, device="cuda:0")
    U = torch.zeros(nova.nova_filter_bytes(K, C, m, nova.NOVA_F16 if dtype == torch.float16 else nova.NOVA_F32, r) // x.element_size(), dtype=dtype, device="cuda:0")
    ws = workspace(t, x, K, 0)
    name = launches(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))[0][0]
    return name.startswith(f"layer_kernel<{t.n}, {r}, half, 16, 64," if dtype == torch.float16 else f"layer_kernel<{t.n}, {r}, float, 16, 32,")


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
def test_64_channels_equal_the_stages(m, r, N, C, K, H, W):
    assert is_wide(m, r, N, C, K, H, W, torch.float16)
    equals_the_stages(m, r, N, C, K, H, W, torch.float16, True)


CASES_BINARY32 = [
    (2, 3, 3, 24, 128, 110, 110), (2, 3, 3, 64, 50, 67, 79), (4, 3, 22, 16, 96, 25, 25), (4, 3, 9, 5, 17, 60, 61), (4, 3, 15, 40, 65, 29, 26),
    (2, 5, 4, 16, 32, 53, 53),
]


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES_BINARY32)
def test_32_channels_of_binary32_equal_the_stages(m, r, N, C, K, H, W):
    assert is_wide(m, r, N, C, K, H, W, torch.float32)
    equals_the_stages(m, r, N, C, K, H, W, torch.float32, True)
