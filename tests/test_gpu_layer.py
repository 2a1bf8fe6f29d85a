"""The whole layer in one kernel (calls with little work) against the separate stage calls: the same operations in
the same order, so the results are equal bit for bit.  The sizes sit at the edges of its workgroups: 8 tiles (CASES, nearly all)
or 16 (CASES_OF_16_TILES), 16 or 32 output channels, blocks of 32 (binary16) or 16 (binary32) input channels."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # m, r, N, C, K, H, W
    (2, 3, 1, 5, 1, 2, 2), (2, 3, 3, 33, 31, 9, 7), (2, 3, 2, 64, 65, 16, 34),
    (4, 3, 1, 16, 16, 32, 32), (4, 3, 1, 6, 17, 1, 29), (4, 3, 5, 31, 33, 12, 4), (4, 3, 3, 32, 40, 30, 41), (4, 3, 1, 65, 32, 28, 28),
    (4, 3, 1, 64, 128, 112, 112), (4, 3, 1, 100, 64, 28, 28),
    (6, 3, 2, 40, 70, 45, 61), (6, 3, 8, 64, 64, 56, 56), (6, 3, 3, 64, 32, 14, 18), (6, 3, 1, 15, 48, 6, 50), (6, 3, 9, 17, 5, 7, 6),
    (8, 3, 1, 11, 82, 25, 12), (8, 3, 2, 64, 32, 24, 40), (8, 3, 9, 48, 15, 8, 8), (8, 3, 1, 7, 33, 3, 3),
    (2, 5, 2, 20, 40, 17, 18), (4, 5, 4, 48, 96, 35, 35), (4, 5, 1, 9, 16, 4, 5), (6, 5, 3, 28, 42, 34, 24), (6, 5, 1, 33, 17, 13, 7),
]

F16, F32 = torch.float16, torch.float32
CASES_OF_16_TILES = [
    # as the rule has it on 256 compute units: 16 q + 1 and 16 q + 15 tiles of every kernel, the listed 5 x 5 workload, and
    # 64 input channels of F(6,3) in binary16, whose outputs are transformed rows first
    (2, 3, 19, 6, 33, 49, 5, F16), (2, 3, 11, 5, 16, 53, 14, F16), (2, 3, 11, 8, 33, 5, 65, F32), (2, 3, 7, 17, 33, 13, 30, F32),
    (4, 3, 17, 12, 33, 19, 51, F16), (4, 3, 11, 5, 16, 49, 68, F16), (4, 3, 17, 5, 17, 19, 52, F32), (4, 3, 9, 10, 96, 52, 10, F32),
    (2, 5, 11, 12, 33, 66, 5, F16), (2, 5, 7, 12, 16, 21, 53, F16), (2, 5, 7, 9, 33, 29, 18, F32), (2, 5, 9, 9, 17, 34, 13, F32),
    (6, 3, 11, 6, 33, 65, 51, F16), (6, 3, 17, 18, 48, 53, 37, F16), (6, 3, 17, 5, 64, 66, 14, F32), (6, 3, 13, 14, 96, 13, 49, F32),
    (4, 5, 5, 11, 33, 68, 49, F16), (4, 5, 19, 5, 17, 34, 51, F16), (4, 5, 17, 5, 64, 42, 9, F32), (4, 5, 15, 8, 33, 25, 25, F32),
    (2, 3, 9, 5, 32, 90, 90, F16), (4, 3, 2, 256, 64, 121, 124, F16), (4, 3, 30, 8, 20, 75, 66, F16), (6, 3, 32, 70, 64, 44, 48, F16),
    (4, 5, 16, 48, 96, 35, 35, F16), (6, 3, 17, 64, 64, 50, 49, F16), (6, 3, 15, 64, 64, 51, 51, F16),
]
# 64 input channels in binary16, 8 tiles, outputs transformed rows first
ROWS_FIRST = [(6, 3, 3, 64, 32, 14, 18, F16), (6, 3, 8, 64, 64, 56, 56, F16), (8, 3, 2, 64, 32, 24, 40, F16), (8, 3, 1, 64, 64, 40, 33, F16)]


def points_for(m, r):
    size = m + r - 3
    return synth.point_set("standard" if size == 2 else "nova", size)


def workspace(t, x, K, flags):
    N, C, H, W = x.shape
    dt = nova.NOVA_F16 if x.dtype == torch.float16 else nova.NOVA_F32
    nbytes = nova.nova_conv2d_workspace_bytes(N, C, H, W, K, t.m, dt, flags, 0, t.r)
    return torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)              # NaN, if anything reads it


def by_stages(t, x, U, K, flags):
    N, C, H, W = x.shape
    dt = nova.NOVA_F16 if x.dtype == torch.float16 else nova.NOVA_F32
    V = nova.nova_input_transform(t, x)
    if nova.nova_conv2d_path(t, C, H, W, K, dt, flags) == nova.NOVA_PATH_FUSED_OUTPUT:
        return nova.nova_contract_output_fused(t, U, V, N, C, H, W, K, flags=flags)
    M = nova.nova_contract(t, U, V, N, C, H, W, K, flags)
    return nova.nova_output_transform(t, M, N, K, H, W, x.dtype, flags)


def equals_the_stages(m, r, N, C, K, H, W, dtype, one_kernel):
    t = nova.nova_make_transforms(points_for(m, r), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m * 1000 + C)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).to(dtype))
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_POOL2, nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_M_F16):
        if flags & nova.NOVA_FLAG_POOL2 and (H % 2 or W % 2):
            continue
        if flags & nova.NOVA_FLAG_M_F16 and dtype != torch.float16:
            continue
        want = by_stages(t, x, U, K, flags)
        ws = workspace(t, x, K, flags)
        guard = torch.full((want.numel() + 64,), float("nan"), dtype=dtype, device=DEV)
        got = guard[32:32 + want.numel()].view(want.shape)
        nova.nova_winograd_conv2d(t, x, U, K, y=got, flags=flags, workspace=ws)
        torch.cuda.synchronize()
        if one_kernel:
            assert bool((ws == 0xFF).all()), "not the one-kernel path"
        assert torch.isfinite(want).all() and torch.equal(got, want), (dtype, flags)
        assert guard[:32].isnan().all() and guard[-32:].isnan().all()


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_equals_the_stages(m, r, N, C, K, H, W, dtype):
    # C: certainly little work (with more channels the rule may go either way)
    equals_the_stages(m, r, N, C, K, H, W, dtype, C <= (40 if dtype == torch.float16 else 28))


@pytest.mark.parametrize("m,r,N,C,K,H,W,dtype", CASES_OF_16_TILES + ROWS_FIRST)
def test_equals_the_stages_in_one_kernel(m, r, N, C, K, H, W, dtype):
    equals_the_stages(m, r, N, C, K, H, W, dtype, True)


def test_unaligned_operands_and_results():
    # x and y one element off their alignment: window rows and result rows at any element
    for dtype in (torch.float16, torch.float32):
        t = nova.nova_make_transforms(points_for(6, 3), 6, 3)
        N, C, K, H, W = 3, 20, 24, 17, 23
        gen = torch.Generator(device=DEV).manual_seed(5)
        x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
        U = nova.nova_filter_transform(t, (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * 0.1).to(dtype))
        want = by_stages(t, x, U, K, 0)
        xs = torch.zeros(x.numel() + 1, dtype=dtype, device=DEV)[1:].view(x.shape)
        xs.copy_(x)
        ys = torch.zeros(want.numel() + 1, dtype=dtype, device=DEV)[1:].view(want.shape)
        nova.nova_winograd_conv2d(t, xs, U, K, y=ys)
        torch.cuda.synchronize()
        assert torch.equal(ys, want)


def test_output_over_the_input():
    # y == x worked while the separate kernels had read x before they wrote y; it still does
    t = nova.nova_make_transforms(points_for(4, 3), 4, 3)
    gen = torch.Generator(device=DEV).manual_seed(6)
    x = torch.randn((2, 16, 20, 20), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((16, 16, 3, 3), device=DEV, generator=gen) * 0.1).half())
    want = nova.nova_winograd_conv2d(t, x, U, 16)
    nova.nova_winograd_conv2d(t, x, U, 16, y=x)
    torch.cuda.synchronize()
    assert torch.equal(x, want)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("m,C,K", [(4, 20, 24), (6, 64, 32), (8, 20, 24)])
def test_values_that_are_not_finite(bad, m, C, K):
    t = nova.nova_make_transforms(points_for(m, 3), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(7)
    for dtype in (torch.float16, torch.float32):
        x = torch.randn((2, C, 20, 22), device=DEV, generator=gen).to(dtype)
        x[1, 3, 7, 9] = bad
        U = nova.nova_filter_transform(t, (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * 0.1).to(dtype))
        for flags in (0, nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_POOL2):
            want, got = by_stages(t, x, U, K, flags), nova.nova_winograd_conv2d(t, x, U, K, flags=flags)
            torch.cuda.synchronize()
            assert torch.equal(got.nan_to_num(nan=7.0), want.nan_to_num(nan=7.0)) and not torch.isfinite(got).all()


@pytest.mark.parametrize("m,r,dtype,N,C,K,H,W", [(6, 5, torch.float16, 13, 97, 512, 4, 4), (2, 3, torch.float16, 5, 416, 320, 12, 12),
                                                 (6, 5, torch.float32, 4, 36, 361, 6, 68), (2, 3, torch.float32, 33, 352, 128, 4, 4)])
def test_faster_as_separate_kernels(m, r, dtype, N, C, K, H, W):
    # few tiles in many rows of M that are never written, or many blocks of input channels: 1.2 to 1.3 times as long as one kernel
    t = nova.nova_make_transforms(points_for(m, r), m, r)
    x = torch.ones((N, C, H, W), device=DEV, dtype=dtype)
    U = nova.nova_filter_transform(t, torch.ones((K, C, r, r), device=DEV, dtype=dtype) / C)
    ws = workspace(t, x, K, 0)
    nova.nova_winograd_conv2d(t, x, U, K, workspace=ws)
    assert (ws != 0xFF).any()


def pooled_as_stated(y):
    # the first of the largest in the order of the image: a zero keeps the sign that the first zero had
    a = y.float().cpu()
    best = a[..., 0::2, 0::2]
    for v in (a[..., 0::2, 1::2], a[..., 1::2, 0::2], a[..., 1::2, 1::2]):
        best = torch.where(v > best, v, best)
    return best.to(y.dtype)


@pytest.mark.parametrize("m,C,K,N,H,W", [(4, 20, 24, 2, 20, 22), (6, 64, 32, 2, 20, 22), (8, 20, 24, 1, 18, 26),          # one kernel
                                         (6, 64, 64, 8, 112, 112), (8, 64, 32, 4, 200, 168),                             # fused 64-channel kernel
                                         (4, 3, 40, 2, 30, 26), (8, 3, 40, 2, 30, 26),                                   # first layer
                                         (8, 128, 64, 120, 32, 40), (8, 300, 64, 8, 48, 48)])                             # columns; separate kernels
def test_signs_of_zeros_under_pooling(m, C, K, N, H, W):
    # results so small that binary16 rounds most of them to a zero, of either sign
    t = nova.nova_make_transforms(points_for(m, 3), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(31 * m + C)
    x = (torch.randn((N, C, H, W), device=DEV, generator=gen) * 2.0 ** -8).half()
    w = (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * 2.0 ** -17 / (9.0 * C) ** 0.5).half()
    U = nova.nova_filter_transform(t, w)
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_M_F16, nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_M_F16):
        plain = nova.nova_winograd_conv2d(t, x, U, K, flags=flags)
        want = pooled_as_stated(plain).view(torch.int16)
        got = nova.nova_winograd_conv2d(t, x, U, K, flags=flags | nova.NOVA_FLAG_POOL2).cpu().view(torch.int16)
        assert (want == 0).any() and (want > 0).any() and (flags & nova.NOVA_FLAG_RELU or (want == -32768).any())
        assert torch.equal(got, want), (flags, int((got != want).sum()))
        if C > 4:
            assert torch.equal(by_stages(t, x, U, K, flags | nova.NOVA_FLAG_POOL2).cpu().view(torch.int16), want), flags
