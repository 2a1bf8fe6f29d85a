"""The output transform's store variants: images of several tile groups per row (even, vectorisable and sector-aligned
group widths, ragged last groups), images that share a workgroup, and rows moved to LDS in pieces -- against
A^T M A evaluated in binary64 on the M the kernel was given."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # m, r, N, K, H, W: several groups per row (17, 28, 38, 56 tiles), W a whole number of pieces or not
    (8, 3, 1, 33, 16, 136), (8, 3, 1, 5, 24, 224), (6, 3, 1, 33, 12, 224), (6, 3, 2, 32, 7, 112), (4, 3, 1, 40, 8, 224),
    (4, 3, 1, 3, 12, 100), (2, 3, 1, 33, 6, 120), (2, 3, 1, 2, 4, 70), (8, 3, 1, 8, 9, 141), (6, 5, 1, 33, 13, 152), (4, 5, 1, 7, 5, 97),
    # one to four tiles per image, image counts that leave the last workgroup ragged
    (8, 3, 17, 65, 7, 7), (8, 3, 515, 32, 8, 8), (8, 3, 9, 40, 14, 14), (6, 3, 7, 33, 6, 12), (4, 3, 300, 64, 4, 3), (2, 5, 11, 34, 2, 4),
    (8, 3, 1024, 33, 16, 8), (6, 3, 700, 32, 10, 10),
]


@pytest.mark.parametrize("m,r,N,K,H,W", CASES)
def test_output_transform_groups(m, r, N, K, H, W):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    n, th, tw = t.n, -(-H // m), -(-W // m)
    T = N * th * tw
    Tp, kb = -(-T // 128) * 128, -(-K // 32)
    A = torch.tensor(nova.nova_get_matrix_f32(t, nova.NOVA_MATRIX_A), dtype=torch.float64, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(W + N)
    M32 = torch.randn((n * n, kb, Tp, 32), device=DEV, generator=gen)
    for dtype, flags in ((torch.float16, 0), (torch.float16, nova.NOVA_FLAG_M_F16 | nova.NOVA_FLAG_RELU), (torch.float32, 0)):
        print(f"[case] output transform F({m},{r}) {dtype} flags {flags} N={N} K={K} {H}x{W}", flush=True)
        M = M32.half() if flags & nova.NOVA_FLAG_M_F16 else M32
        P = M[:, :, :T].double().permute(0, 2, 1, 3).reshape(n, n, T, kb * 32)[:, :, :, :K]

        def through(a, p):
            z = torch.tensordot(a, torch.tensordot(a, p, dims=([0], [0])), dims=([0], [1]))         # [q, p, T, K]
            return z.reshape(m, m, N, th, tw, K).permute(2, 5, 3, 1, 4, 0).reshape(N, K, th * m, tw * m)[:, :, :H, :W]

        want, size_of = through(A, P), through(A.abs(), P.abs())
        if flags & nova.NOVA_FLAG_RELU:
            want = want.clamp(min=0.0)
        # 2 n roundings of binary32 at most of the absolute sum, then one to the storage format
        bound = 2 * (2 * n + 2) * 2.0 ** -24 * size_of + (2.0 ** -11 * want.abs() + 2.0 ** -25 if dtype == torch.float16 else 0.0)
        for pool in (False, True) if H % 2 == 0 and W % 2 == 0 else (False,):
            got = torch.full((N, K) + ((H // 2, W // 2) if pool else (H, W)), float("nan"), dtype=dtype, device=DEV)
            nova.nova_output_transform(t, M.reshape(-1), N, K, H, W, dtype, flags | (nova.NOVA_FLAG_POOL2 if pool else 0), y=got)
            if pool:
                assert torch.equal(got.float(), torch.nn.functional.max_pool2d(plain.float(), 2))
            else:
                assert ((got.double() - want).abs() <= bound).all(), float(((got.double() - want).abs() / bound).max())
                plain = got
