"""Calls whose products leave the contraction with their columns transformed (m planes of n instead of M) against the
separate stage calls: the same operations in the same order, so the results are equal bit for bit.  The sizes sit at the
edges of its 64 x 64 (one block of output channels: 128 x 32) tiles and of its channel loop.  Where contraction and output run as one kernel or the
layer does (n = 4; 5 x 5 and F(4,3) of fewer channels), calls whose y lies over x still come here.  The launched kernels are asserted."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # m, r, N, C, K, H, W
    (4, 3, 9, 200, 100, 61, 62), (6, 3, 17, 96, 130, 45, 47), (6, 3, 6, 200, 256, 60, 65), (6, 3, 76, 230, 32, 60, 66),
    (8, 3, 34, 65, 96, 50, 52), (8, 3, 120, 128, 64, 32, 40), (8, 3, 70, 80, 20, 66, 70),
    (2, 5, 10, 160, 64, 33, 50), (4, 5, 20, 140, 96, 35, 35), (6, 5, 70, 20, 64, 30, 40),
]
# with y over x: 64 x 64 tiles of n = 4 and 6, 128 x 32 ones
OVER_X = [(2, 3, 5, 33, 70, 60, 100), (2, 3, 20, 5, 32, 90, 90), (4, 3, 9, 40, 100, 61, 62), (4, 3, 40, 8, 20, 75, 66), (6, 3, 42, 33, 64, 44, 48),
          (2, 5, 10, 100, 64, 33, 50), (2, 5, 12, 40, 30, 70, 70), (4, 5, 20, 48, 96, 35, 35), (4, 5, 20, 30, 32, 66, 66)]


def kernels(call):
    return [name.split("<")[0] for name, _, _ in launches(call)]


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
def test_equals_the_stages(m, r, N, C, K, H, W):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m * 1000 + C)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).half())
    V = nova.nova_input_transform(t, x)
    M = nova.nova_contract(t, U, V, N, C, H, W, K)
    planes = nova.nova_product_bytes(N, K, H, W, m, nova.NOVA_F16, 0, r)
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_POOL2):
        if flags & nova.NOVA_FLAG_POOL2 and (H % 2 or W % 2):
            continue
        want = nova.nova_output_transform(t, M, N, K, H, W, torch.float16, flags)
        nbytes = nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, nova.NOVA_F16, flags, N, r)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)                # NaN, if anything reads it
        got = torch.empty_like(want)
        assert "contract_columns_kernel" in kernels(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=got, flags=flags, workspace=ws))
        nova.nova_winograd_conv2d(t, x, U, K, y=got, flags=flags, workspace=ws)
        some = nova.nova_winograd_conv2d(t, x, U, K, flags=flags, images_per_slab=2)
        torch.cuda.synchronize()
        assert torch.isfinite(want).all() and torch.equal(got, want) and torch.equal(some, want), flags
        tail = planes // t.n * (t.n - m)                                               # the planes that are not written
        assert bool((ws[nbytes - tail:] == 0xFF).all()), "not this path"


@pytest.mark.parametrize("m,r,N,C,K,H,W", OVER_X)
def test_output_over_the_input(m, r, N, C, K, H, W):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m * 1000 + C)
    memory = torch.empty(N * max(C, K) * H * W + 8, dtype=torch.float16, device=DEV)
    x, y = memory[:N * C * H * W].view(N, C, H, W), memory[8:8 + N * K * H * W].view(N, K, H, W)
    start = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    x.copy_(start)
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).half())
    want = nova.nova_output_transform(t, nova.nova_contract(t, U, nova.nova_input_transform(t, start), N, C, H, W, K), N, K, H, W, torch.float16)
    ws = torch.empty(nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, nova.NOVA_F16, 0, N, r), dtype=torch.uint8, device=DEV)
    assert kernels(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))[1] == "contract_columns_kernel"
    nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and torch.equal(y, want)


@pytest.mark.parametrize("N,C,K,H,W", [(19, 256, 256, 44, 44), (16, 256, 512, 65, 9), (7, 128, 384, 43, 43), (11, 192, 384, 40, 44), (32, 227, 128, 85, 15)])
def test_faster_as_separate_kernels(N, C, K, H, W):
    # M is written whole: 1.03 to 1.1 times as long this way
    t = nova.nova_make_transforms(synth.point_set("nova", 6), 6, 3)
    x = torch.ones((N, C, H, W), device=DEV, dtype=torch.float16)
    U = nova.nova_filter_transform(t, torch.ones((K, C, 3, 3), device=DEV, dtype=torch.float16) / C)
    nbytes = nova.nova_conv2d_workspace_bytes(N, C, H, W, K, 6, nova.NOVA_F16, 0, N)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
    nova.nova_winograd_conv2d(t, x, U, K, workspace=ws)
    last = nova.nova_product_bytes(N, K, H, W, 6, nova.NOVA_F16) // 64                     # the last of the 64 planes of M
    assert (ws[nbytes - last:] != 0xFF).any()


def test_slabs_no_larger_than_the_cache():
    # 27 images, 102 MB of x and 230 MB of V, fit the workspace with m of n planes (307 MB), not with M whole (346): two slabs
    t = nova.nova_make_transforms(synth.point_set("nova", 4), 4, 3)
    N, C, K, H, W = 27, 256, 64, 44, 168
    x = torch.ones((N, C, H, W), device=DEV, dtype=torch.float16)
    y = torch.empty((N, K, H, W), device=DEV, dtype=torch.float16)
    U = nova.nova_filter_transform(t, torch.ones((K, C, 3, 3), device=DEV, dtype=torch.float16) / C)
    ws = torch.empty(310_000_000, dtype=torch.uint8, device=DEV)
    v, m_whole = nova.nova_input_bytes(N, C, H, W, 4, nova.NOVA_F16), nova.nova_product_bytes(N, K, H, W, 4, nova.NOVA_F16)
    assert v + m_whole // 6 * 4 + 512 <= ws.numel() < v + m_whole and v + x.numel() * 2 > 256 << 20
    assert kernels(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws)) == ["input_transform_kernel", "contract_columns_kernel", "output_transform_kernel"] * 2


def test_values_that_are_not_finite():
    t = nova.nova_make_transforms(synth.point_set("nova", 4), 4, 3)
    gen = torch.Generator(device=DEV).manual_seed(7)
    x = torch.randn((9, 200, 61, 62), device=DEV, generator=gen).half()
    x[1, 3, 7, 9], x[5, 30, 20, 11] = float("inf"), float("nan")
    U = nova.nova_filter_transform(t, (torch.randn((100, 200, 3, 3), device=DEV, generator=gen) * 0.1).half())
    V = nova.nova_input_transform(t, x)
    M = nova.nova_contract(t, U, V, 9, 200, 61, 62, 100)
    want, got = nova.nova_output_transform(t, M, 9, 100, 61, 62, torch.float16), torch.empty((9, 100, 61, 62), dtype=torch.float16, device=DEV)
    ws = torch.empty(nova.nova_conv2d_workspace_bytes(9, 200, 61, 62, 100, 4, nova.NOVA_F16), dtype=torch.uint8, device=DEV)
    assert "contract_columns_kernel" in kernels(lambda: nova.nova_winograd_conv2d(t, x, U, 100, y=got, workspace=ws))
    nova.nova_winograd_conv2d(t, x, U, 100, y=got, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(got.nan_to_num(nan=7.0), want.nan_to_num(nan=7.0)) and not torch.isfinite(got).all()
