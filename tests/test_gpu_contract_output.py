"""Calls that run contraction and output transform as one kernel (32 x 32 tiles and output channels per workgroup, stages of two positions
and 64 input channels) against the separate stage calls: the same operations in the same order, so the results are equal bit
for bit.  Odd and even numbers of channel blocks, partial last tiles and output channels, images of one cropped tile, whose rows leave
through LDS, and wide ones.  The launched kernels are asserted."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # m, r, N, C, K, H, W
    (2, 3, 21, 33, 70, 60, 62), (2, 3, 11, 250, 100, 61, 64), (2, 3, 13, 130, 64, 62, 70),
    (4, 3, 24, 64, 64, 47, 60), (4, 3, 9, 97, 128, 40, 61), (4, 3, 27, 160, 160, 30, 26), (4, 3, 250, 100, 96, 14, 7),
    (6, 3, 40, 40, 96, 46, 50), (6, 3, 30, 128, 130, 48, 49), (6, 3, 3000, 90, 64, 6, 5), (6, 3, 300, 65, 80, 7, 24),
    (2, 5, 12, 70, 40, 61, 50), (4, 5, 16, 48, 96, 44, 52), (4, 5, 50, 120, 64, 30, 22), (6, 5, 70, 60, 100, 30, 40), (6, 5, 100, 128, 128, 25, 36),
    (2, 3, 5, 33, 70, 60, 100), (4, 3, 9, 40, 100, 61, 62), (2, 5, 10, 100, 64, 33, 50), (4, 5, 20, 48, 96, 35, 35),
    # V and y of 372 MB: rows of 12 bytes with the streaming hint; 5 x 5 with an odd number of blocks up to 192 channels
    (6, 3, 420, 128, 256, 24, 26), (6, 5, 150, 161, 120, 25, 32),
]


def runs_here(call):
    return all(name.startswith(("input_transform_kernel", "contract_output_kernel")) for name, _, _ in launches(call))


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
def test_equals_the_stages(m, r, N, C, K, H, W):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m * 1000 + C)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).half())
    V = nova.nova_input_transform(t, x)
    M = nova.nova_contract(t, U, V, N, C, H, W, K)
    v_bytes = nova.nova_input_bytes(N, C, H, W, m, nova.NOVA_F16, r)
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_POOL2, nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_POOL2):
        if flags & nova.NOVA_FLAG_POOL2 and (H % 2 or W % 2):
            continue
        want = nova.nova_output_transform(t, M, N, K, H, W, torch.float16, flags)
        nbytes = nova.nova_conv2d_workspace_bytes(N, C, H, W, K, m, nova.NOVA_F16, flags, N, r)
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)                # NaN, if anything reads it
        y = torch.full_like(want, 123.0)
        names = [name for name, _, _ in launches(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, flags=flags, workspace=ws))]
        assert names[1].startswith("contract_output_kernel") and names[1].endswith(", 1>" if (N, C, K) == (420, 128, 256) else ", 0>"), names
        got = nova.nova_winograd_conv2d(t, x, U, K, y=y, flags=flags, workspace=ws)
        torch.cuda.synchronize()
        assert torch.isfinite(want).all() and torch.equal(got, want), flags
        if flags & nova.NOVA_FLAG_POOL2:
            assert torch.equal(torch.signbit(got), torch.signbit(want))
        assert bool((ws[:4096] != 0xFF).any()) and bool((ws[(v_bytes + 255) // 256 * 256:] == 0xFF).all()), "not this path"


def test_slabs_and_replays():
    # four slabs, the last shorter than the others, and the call captured: replays after other work equal the eager call
    t = nova.nova_make_transforms(synth.point_set("nova", 4), 4, 3)
    N, C, K, H, W = 61, 96, 128, 50, 52
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * 0.05).half())
    want = nova.nova_output_transform(t, nova.nova_contract(t, U, nova.nova_input_transform(t, x), N, C, H, W, K), N, K, H, W, torch.float16)
    v_image = nova.nova_input_bytes(1, C, H, W, 4, nova.NOVA_F16)
    ws = torch.empty(17 * v_image + 256, dtype=torch.uint8, device=DEV)                # 61 images: 16, 16, 16 and 13
    y = torch.empty_like(want)
    assert [blocks for _, blocks, _ in launches(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))][1::2] == [16 * 169 // 32 * 4 + 4] * 3 + [13 * 169 // 32 * 4 + 4]
    assert runs_here(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))
    nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws)
    for _ in range(3):
        y.fill_(7.0)
        ws.fill_(0xFF)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


def test_values_that_are_not_finite():
    t = nova.nova_make_transforms(synth.point_set("nova", 6), 6, 3)
    gen = torch.Generator(device=DEV).manual_seed(7)
    x = torch.randn((40, 40, 46, 50), device=DEV, generator=gen).half()
    x[1, 3, 7, 9], x[5, 30, 20, 11], x[9, 2, 45, 49] = float("inf"), float("nan"), float("-inf")
    U = nova.nova_filter_transform(t, (torch.randn((96, 40, 3, 3), device=DEV, generator=gen) * 0.1).half())
    M = nova.nova_contract(t, U, nova.nova_input_transform(t, x), 40, 40, 46, 50, 96)
    ws = torch.empty(nova.nova_conv2d_workspace_bytes(40, 40, 46, 50, 96, 6, nova.NOVA_F16), dtype=torch.uint8, device=DEV)
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_POOL2):
        want = nova.nova_output_transform(t, M, 40, 96, 46, 50, torch.float16, flags)
        got = torch.empty_like(want)
        assert runs_here(lambda: nova.nova_winograd_conv2d(t, x, U, 96, y=got, flags=flags, workspace=ws))
        nova.nova_winograd_conv2d(t, x, U, 96, y=got, flags=flags, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got.nan_to_num(nan=7.0), want.nan_to_num(nan=7.0)) and not torch.isfinite(got).all()
