"""Layers of at most 4 input channels in binary16: the kernel that forms the products itself (16 tiles x 32 output channels
per workgroup, two waves sharing the output rows) against the separate stages, whose products come from another matrix
instruction: they agree to rounding."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # m, r, N, C, K, H, W: 1, 15, 16, 17, 33 tiles; one, 31, 32, 33, 65 output channels; ragged rows and columns
    (2, 3, 1, 3, 1, 2, 2), (2, 3, 3, 4, 33, 9, 13), (4, 3, 1, 1, 31, 12, 20), (4, 3, 1, 2, 32, 16, 16), (4, 3, 1, 3, 65, 3, 66),
    (6, 3, 1, 4, 64, 15, 64), (6, 3, 2, 3, 40, 50, 46), (8, 3, 1, 3, 64, 8, 8), (8, 3, 1, 2, 33, 24, 40), (8, 3, 3, 3, 5, 31, 26),
    (8, 3, 2, 4, 64, 64, 72), (2, 5, 2, 3, 20, 17, 6), (4, 5, 1, 4, 48, 20, 23), (6, 5, 2, 1, 34, 19, 44),
]


@pytest.mark.parametrize("m,r,N,C,K,H,W", CASES)
def test_agrees_with_the_stages(m, r, N, C, K, H, W):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(100 * m + C)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5).half())
    V = nova.nova_input_transform(t, x)
    # Two binary32 summations of at most 4 products: y differs where its rounding to binary16 falls to the other side,
    # by one unit in the last place (2^-11 relative) in few elements; with products rounded to binary16 a product
    # does so, which n = 10 amplifies as it amplifies any other rounding (bar of the emulation: 5e-3)
    for products16 in (0, nova.NOVA_FLAG_M_F16):
        M = nova.nova_contract(t, U, V, N, C, H, W, K, products16)
        want = nova.nova_output_transform(t, M, N, K, H, W, torch.float16, products16)
        guard = torch.full((want.numel() + 65,), float("nan"), dtype=torch.float16, device=DEV)
        got = guard[33:33 + want.numel()].view(want.shape)                 # one element off its alignment
        nova.nova_winograd_conv2d(t, x, U, K, y=got, flags=products16)
        relu = nova.nova_winograd_conv2d(t, x, U, K, flags=products16 | nova.NOVA_FLAG_RELU)
        torch.cuda.synchronize()
        assert torch.isfinite(got).all() and guard[:33].isnan().all() and guard[-32:].isnan().all()
        err = ((got.double() - want.double()).norm() / want.double().norm()).item()
        assert err < (1e-3 if not products16 or m + r < 11 else 2e-2), err
        assert torch.equal(relu, torch.clamp(got, min=0))
        if H % 2 == 0 and W % 2 == 0:
            pooled = nova.nova_winograd_conv2d(t, x, U, K, flags=products16 | nova.NOVA_FLAG_RELU | nova.NOVA_FLAG_POOL2)
            torch.cuda.synchronize()
            assert torch.equal(pooled.float(), torch.nn.functional.max_pool2d(relu.float(), 2))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_values_that_are_not_finite(bad):
    # a pixel that is not finite spoils the outputs of its tiles' neighbourhood and nothing else
    t = nova.nova_make_transforms(synth.point_set("nova", 6), 6, 3)
    gen = torch.Generator(device=DEV).manual_seed(8)
    x = torch.randn((2, 3, 40, 52), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((40, 3, 3, 3), device=DEV, generator=gen) * 0.2).half())
    clean = nova.nova_winograd_conv2d(t, x, U, 40)
    x[1, 2, 20, 33] = bad
    V = nova.nova_input_transform(t, x)
    stages = nova.nova_output_transform(t, nova.nova_contract(t, U, V, 2, 3, 40, 52, 40), 2, 40, 40, 52, torch.float16)
    for flags in (0, nova.NOVA_FLAG_RELU):
        got = nova.nova_winograd_conv2d(t, x, U, 40, flags=flags)
        torch.cuda.synchronize()
        same = torch.isfinite(stages)
        want = torch.clamp(clean, min=0) if flags else clean
        assert torch.equal(got[same], want[same])
        assert got.isnan().any() and (flags or not torch.isfinite(got[~same]).any())


@pytest.mark.parametrize("scale_x,scale_w", [(2.0 ** -24, 1.0), (1.0, 2.0 ** -24)])
@pytest.mark.parametrize("C,W", [(3, 25), (4, 70)])
def test_subnormal_operands(scale_x, scale_w, C, W):
    # F(2,3) with points 0, 1, -1 and filters in multiples of 4: V, U, every product, partial sum and result is a whole
    # multiple of 2^-24 below 2^11 of them, exact in binary16 (V or U subnormal), so nothing may be flushed to zero
    t = nova.nova_make_transforms(synth.point_set("standard", 2), 2, 3)
    gen = torch.Generator(device=DEV).manual_seed(C)
    x = torch.randint(-13, 14, (2, C, 21, W), device=DEV, generator=gen).double()
    w = 4.0 * torch.randint(-1, 2, (35, C, 3, 3), device=DEV, generator=gen).double()
    want = torch.nn.functional.conv2d(x.cpu(), w.cpu(), padding=1) * (scale_x * scale_w)
    U = nova.nova_filter_transform(t, (w * scale_w).half())
    y = nova.nova_winograd_conv2d(t, (x * scale_x).half(), U, 35)
    torch.cuda.synchronize()
    assert want.abs().max() < 2.0 ** -13 and (want != 0).any() and torch.equal(y.double().cpu(), want)
