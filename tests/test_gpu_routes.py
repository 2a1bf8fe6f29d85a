"""Which kernel leaves the results of layers that measured faster with it than with another that takes such layers, at sizes well inside
the rules.  The kernels are read from a captured graph that never runs; that all of them give the same bits is tested elsewhere."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F16, F32 = torch.float16, torch.float32

# m, r, N, C, K, H, W, type, kernel
ROUTES = [
    # F(2,3) with few output channels and workgroups enough for contraction and output in one kernel: the whole layer in one is faster (15.9 / 21.4 us,
    # 10.3 / 17.0, 10.4 / 17.2, 11.7 / 13.1); with more of either it is not (22.2 / 23.6, 39.7 / 44.5)
    (2, 3, 71, 64, 64, 23, 24, F16, "layer_kernel"), (2, 3, 2309, 48, 33, 2, 6, F16, "layer_kernel"), (2, 3, 674, 64, 33, 6, 7, F16, "layer_kernel"),
    (2, 3, 41, 24, 64, 34, 31, F16, "layer_kernel"), (2, 3, 48, 64, 192, 23, 22, F16, "contract_output_kernel"),
    (2, 3, 53, 128, 128, 31, 28, F16, "contract_output_kernel"),
    # 16 tiles with 64 output channels only where that saves a round of workgroups that takes as long: 7.8 / 10.0 us, 7.8 / 8.3 with 32; 19.0 / 15.2 with 64
    (2, 3, 14, 80, 64, 19, 22, F16, "layer_kernel<4, 3, half, 16, 32,"), (2, 3, 6, 48, 256, 21, 24, F16, "layer_kernel<4, 3, half, 16, 32,"),
    (2, 3, 27, 24, 64, 34, 33, F16, "layer_kernel<4, 3, half, 16, 64,"),
]


@pytest.mark.parametrize("m,r,N,C,K,H,W,dtype,kernel", ROUTES)
def test_route(m, r, N, C, K, H, W, dtype, kernel):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    x = torch.zeros((N, C, H, W), dtype=dtype, device=DEV)
    y = torch.empty((N, K, H, W), dtype=dtype, device=DEV)
    dt = nova.NOVA_F16 if dtype == F16 else nova.NOVA_F32
    U = torch.zeros(nova.nova_filter_bytes(K, C, m, dt, r) // x.element_size(), dtype=dtype, device=DEV)
    ws = torch.empty(nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, dt, 0, 0, r), dtype=torch.uint8, device=DEV)
    got = launches(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))
    assert got[-1][0].startswith(kernel), got
