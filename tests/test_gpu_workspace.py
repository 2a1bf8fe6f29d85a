"""Slabs, poisoned workspaces and graph capture on layers with too much work for one kernel: their V and M go through the
workspace, which the small layers of test_gpu_parity.py, one kernel each, leave alone.  Ragged tile counts and channels on
every path: three kernels in binary32 and in binary16 (also with products rounded to binary16), columns, the fused 64-channel kernel."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F16, F32 = torch.float16, torch.float32
RELU, M16 = nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_M_F16

CASES = [
    # m, r, N, C, K, H, W, type, flags
    (8, 3, 5, 200, 130, 29, 33, F16, 0), (8, 3, 5, 200, 130, 29, 33, F16, RELU | M16), (8, 3, 7, 256, 128, 28, 30, F16, RELU),
    (6, 3, 5, 300, 70, 27, 56, F16, RELU), (6, 3, 5, 300, 70, 27, 56, F16, M16), (4, 3, 5, 270, 100, 23, 35, F16, 0), (2, 3, 5, 500, 70, 13, 22, F16, RELU),
    (4, 5, 5, 210, 100, 23, 30, F16, 0), (4, 3, 5, 170, 50, 19, 22, F32, RELU), (8, 3, 5, 150, 90, 19, 25, F32, 0), (6, 3, 5, 170, 65, 31, 20, F32, 0),
    (4, 3, 9, 200, 160, 61, 62, F16, RELU),                   # columns (in one slab)
    (6, 3, 13, 64, 96, 61, 77, F16, RELU), (8, 3, 13, 64, 160, 61, 77, F16, 0),                # fused
]


def layer(m, r, N, C, K, H, W, dtype):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(1000 * m + C)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
    return t, x, nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).to(dtype))


@pytest.mark.parametrize("m,r,N,C,K,H,W,dtype,flags", CASES)
def test_slabs_and_poisoned_workspaces(m, r, N, C, K, H, W, dtype, flags):
    # Workspace and y are NaN before the call; the same bits come out whatever the slabs
    t, x, U = layer(m, r, N, C, K, H, W, dtype)
    dt = nova.NOVA_F16 if dtype == F16 else nova.NOVA_F32
    V = nova.nova_input_transform(t, x)
    if nova.nova_conv2d_path(t, C, H, W, K, dt, flags) == nova.NOVA_PATH_FUSED_OUTPUT:
        want = nova.nova_contract_output_fused(t, U, V, N, C, H, W, K, flags=flags)
    else:
        want = nova.nova_output_transform(t, nova.nova_contract(t, U, V, N, C, H, W, K, flags), N, K, H, W, dtype, flags)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    for per_slab in (N, 2, 1):
        dirty = torch.full((nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, dt, flags, per_slab, r),), 0xFF, dtype=torch.uint8, device=DEV)
        got = torch.full_like(want, float("nan"))
        nova.nova_winograd_conv2d(t, x, U, K, y=got, flags=flags, workspace=dirty)
        torch.cuda.synchronize()
        assert torch.equal(got, want), per_slab
        assert (dirty != 0xFF).any(), "one kernel: not what is tested here"
    with pytest.raises(nova.NovaError) as exc:
        nova.nova_winograd_conv2d(t, x, U, K, flags=flags, workspace=dirty[:nova.nova_input_bytes(1, C, H, W, m, dt, r) - 1])       # V alone does not fit
    assert exc.value.code == -5
    torch.cuda.synchronize()


@pytest.mark.parametrize("m,r,N,C,K,H,W,dtype,flags", CASES[::3])
def test_graph_of_several_kernels(m, r, N, C, K, H, W, dtype, flags):
    t, x, U = layer(m, r, N, C, K, H, W, dtype)
    dt = nova.NOVA_F16 if dtype == F16 else nova.NOVA_F32
    ws = torch.full((nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, dt, flags, 2, r),), 0xFF, dtype=torch.uint8, device=DEV)
    y = nova.nova_winograd_conv2d(t, x, U, K, flags=flags, workspace=ws)                    # warm up outside the capture
    torch.cuda.synchronize()
    assert (ws != 0xFF).any()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nova.nova_winograd_conv2d(t, x, U, K, y=y, flags=flags, workspace=ws)
    gen = torch.Generator(device=DEV).manual_seed(3)
    for rep in range(3):
        x.copy_(torch.randn(x.shape, device=DEV, generator=gen).to(dtype))
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = nova.nova_winograd_conv2d(t, x, U, K, flags=flags)
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.isfinite(y).all(), rep
