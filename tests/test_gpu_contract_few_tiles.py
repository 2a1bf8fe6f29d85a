"""Contraction of few tiles with long channel loops (64 x 64 tiles, a ring of five stages, where a launch has few workgroups) against
binary64 sums of the stored U and V; the bound is that of C exact products added in binary32, twice the standard one."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,N,C,K,H", [(4, 1, 512, 512, 14), (4, 1, 225, 70, 28), (4, 1, 300, 129, 5), (8, 64, 256, 512, 7), (8, 65, 240, 512, 7), (8, 3, 512, 512, 7),
                                       (6, 1, 512, 320, 18)])
def test_products(m, N, C, K, H):
    t = nova.nova_make_transforms(synth.point_set("nova", m), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(C + K)
    n2, T, Kp, cb = t.n * t.n, N * (-(-H // m)) ** 2, -(-K // 32) * 32, -(-C // 32)
    V = torch.randn((n2, T, cb * 32), device=DEV, generator=gen).half()
    U = (torch.randn((n2, Kp, cb * 32), device=DEV, generator=gen) * C ** -0.5).half()
    V[:, :, C:], U[:, :, C:], U[:, K:] = 0, 0, 0
    blocked = [a.view(n2, rows, cb, 32).transpose(1, 2).contiguous().view(-1) for a, rows in ((U, Kp), (V, T))]
    M = nova.nova_contract(t, blocked[0], blocked[1], N, C, H, H, K)
    M = M.view(n2, Kp // 32, -(-T // 128) * 128, 32).transpose(1, 2).reshape(n2, -1, Kp)[:, :T, :K].double()
    want = torch.matmul(V.double(), U.double().transpose(1, 2).contiguous())[:, :, :K]
    size = torch.matmul(V.double().abs(), U.double().abs().transpose(1, 2).contiguous())[:, :, :K]
    assert ((M - want).abs() <= 2 * (C + 2) * 2.0 ** -24 * size).all()
