"""Results that leave through LDS (images of few columns; the fused 64-channel kernel and the first layer's) against those that
leave straight from registers: the same image with columns of zeros behind it is a wide one, and zeros are what lies beyond
the border anyway, so the results in the image's columns are the same bits."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def transforms(m, r):
    size = m + r - 3
    return nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)


def compare(call, x, K, flags):
    N, C, H, W = x.shape
    wide = torch.zeros((N, C, H, 96), dtype=x.dtype, device=DEV)
    wide[..., :W] = x
    guard = torch.full((N * K * H * W + 65,), float("nan"), dtype=torch.float16, device=DEV)
    got = guard[33:-32].view(N, K, H, W)                                    # one element off its alignment
    call(x, got, flags)
    want = call(wide, torch.empty((N, K, H, 96), dtype=torch.float16, device=DEV), flags)[..., :W]
    torch.cuda.synchronize()
    assert guard[:33].isnan().all() and guard[-32:].isnan().all() and torch.isfinite(want).all()
    assert torch.equal(got.view(torch.int16), want.contiguous().view(torch.int16)), (flags, (got != want).sum().item())


# tiles: 1, 15, 16, 17, 33 and several images; one to four per row, whole and cut off at either edge
@pytest.mark.parametrize("m,N,K,H,W", [(6, 1, 32, 1, 1), (6, 1, 64, 85, 5), (6, 2, 96, 48, 6), (6, 1, 32, 97, 3), (6, 5, 64, 20, 12), (6, 3, 32, 31, 17),
                                       (6, 2, 224, 14, 24), (6, 2, 32, 23, 25),
                                       (8, 1, 32, 2, 2), (8, 1, 64, 117, 7), (8, 2, 96, 64, 8), (8, 1, 32, 129, 5), (8, 5, 64, 20, 9), (8, 3, 32, 31, 16),
                                       (8, 2, 224, 14, 23), (8, 2, 64, 33, 24)])
def test_fused_kernel(m, N, K, H, W):
    t = transforms(m, 3)
    gen = torch.Generator(device=DEV).manual_seed(W * 100 + m)
    x = torch.randn((N, 64, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, 64, 3, 3), device=DEV, generator=gen) * 0.06).half())

    def call(x, y, flags):
        n, c, h, w = x.shape
        return nova.nova_contract_output_fused(t, U, nova.nova_input_transform(t, x), n, c, h, w, K, flags=flags, y=y)
    for flags in (0, nova.NOVA_FLAG_RELU):
        compare(call, x, K, flags)


@pytest.mark.parametrize("m,r,N,C,K,H,W", [(2, 3, 1, 3, 1, 2, 1), (2, 3, 3, 4, 33, 9, 13), (2, 3, 2, 3, 64, 31, 39), (4, 3, 1, 1, 31, 60, 4), (4, 3, 2, 3, 65, 33, 7),
                                           (4, 3, 4, 3, 32, 20, 39), (6, 3, 1, 4, 64, 91, 5), (6, 3, 2, 3, 40, 50, 12), (6, 3, 7, 2, 5, 8, 29),
                                           (8, 3, 1, 3, 64, 8, 8), (8, 3, 1, 2, 33, 130, 3), (8, 3, 3, 3, 7, 31, 16), (8, 3, 2, 4, 64, 40, 39),
                                           (2, 5, 2, 3, 20, 17, 5), (4, 5, 3, 4, 48, 20, 23), (6, 5, 2, 1, 34, 19, 33)])
def test_first_layer(m, r, N, C, K, H, W):
    t = transforms(m, r)
    gen = torch.Generator(device=DEV).manual_seed(W * 100 + m)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).half())

    def call(x, y, flags):
        return nova.nova_winograd_conv2d(t, x, U, K, y=y, flags=flags)
    for flags in (0, nova.NOVA_FLAG_RELU, nova.NOVA_FLAG_M_F16):
        compare(call, x, K, flags)


def test_rows_of_12_bytes_with_and_without_the_streaming_hint():
    # F(6,3): V and y of the batch exceed the last-level cache (stores with the hint), those of one image do not
    t = transforms(6, 3)
    N, K, H, W = 62, 64, 112, 110
    gen = torch.Generator(device=DEV).manual_seed(12)
    x = torch.randn((N, 64, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, 64, 3, 3), device=DEV, generator=gen) * 0.06).half())
    V = nova.nova_input_transform(t, x)
    y = nova.nova_contract_output_fused(t, U, V, N, 64, H, W, K)
    assert V.numel() * V.element_size() + y.numel() * 2 > 256 << 20
    for i in (0, 30, 61):
        one = nova.nova_contract_output_fused(t, U, nova.nova_input_transform(t, x[i:i + 1].contiguous()), 1, 64, H, W, K)
        torch.cuda.synchronize()
        assert torch.equal(one[0].view(torch.int16), y[i].view(torch.int16))
