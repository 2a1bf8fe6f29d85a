"""The products do not depend on which contraction kernel or tile shape formed them: every variant the dispatch can
choose (by channels, output channels and number of products) against binary64 sums of the stored U and V, and bit for
bit against the same images contracted in small slabs, which run the small tiles."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # m, N, C, K, H, W: 128 x 32 tiles; 64 x 64 with ragged edges both ways, one to many channel blocks
    (4, 1, 5, 32, 9, 9), (4, 3, 33, 20, 45, 50), (6, 2, 31, 33, 31, 33), (4, 1, 64, 64, 32, 32), (4, 1, 97, 129, 33, 31),
    (4, 1, 512, 512, 14, 14), (6, 5, 300, 96, 30, 30),
    # 128 x 64 tiles by the number of products, 128 x 128 by the length of the channel loop
    (4, 9, 48, 96, 140, 140), (8, 15, 260, 260, 20, 20),
    # long channel loops with 64 output channels or fewer
    (8, 15, 260, 64, 20, 20), (8, 25, 260, 50, 40, 40), (4, 64, 257, 33, 45, 45),
    # streaming kernel at its thresholds: C = 256, 128, 64; K a multiple of 256 or of 128 only
    (8, 12, 256, 256, 49, 50), (8, 21, 256, 128, 50, 50), (8, 18, 128, 256, 57, 56), (8, 36, 128, 128, 56, 57),
    (4, 6, 64, 256, 170, 180), (4, 12, 64, 128, 170, 180),
]


def unblock(a, n2, rows, chans):
    return a.view(n2, -(-chans // 32), rows, 32).transpose(1, 2).reshape(n2, rows, -1)[:, :, :chans]


@pytest.mark.parametrize("m,N,C,K,H,W", CASES)
def test_products(m, N, C, K, H, W):
    t = nova.nova_make_transforms(synth.point_set("nova", m), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(C + K)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * (2.0 / (9 * C)) ** 0.5).half())
    n2, per = t.n * t.n, -(-H // m) * -(-W // m)
    T, Kp = N * per, -(-K // 32) * 32
    V = nova.nova_input_transform(t, x)
    Ul, Vl = unblock(U, n2, Kp, C)[:, :K].double(), unblock(V, n2, T, C)
    parts = [nova.nova_input_transform(t, x[i:i + 1].contiguous()) for i in range(min(N, 3))]
    for flags in (0, nova.NOVA_FLAG_M_F16):
        print(f"[case] products F({m},3) N={N} C={C} K={K} {H}x{W} flags={flags}", flush=True)
        M = nova.nova_contract(t, U, V, N, C, H, W, K, flags)
        M = unblock(M, n2, -(-T // 128) * 128, K)[:, :T]
        for i, v in enumerate(parts):
            one = unblock(nova.nova_contract(t, U, v, 1, C, H, W, K, flags), n2, -(-per // 128) * 128, K)[:, :per]
            assert torch.equal(M[:, i * per:(i + 1) * per], one)
        for xi in (0, n2 // 2 + 1, n2 - 1):
            want = torch.matmul(Vl[xi].double(), Ul[xi].t().contiguous())
            size = torch.matmul(Vl[xi].double().abs(), Ul[xi].t().abs().contiguous())
            # C exact products added in binary32 (twice the standard bound, for sums that are truncated), then one rounding
            bound = 2 * (C + 2) * 2.0 ** -24 * size + (2.0 ** -11 * want.abs() + 2.0 ** -25 if flags else 0.0)
            assert ((M[xi].double() - want).abs() <= bound).all(), xi


@pytest.mark.parametrize("m,N,C,K,H,W", [(4, 1, 1, 1, 5, 5), (4, 1, 8, 32, 33, 32), (2, 2, 9, 33, 13, 21), (6, 3, 32, 64, 49, 31),
                                         (4, 2, 41, 65, 32, 65), (6, 2, 160, 96, 25, 60), (8, 1, 64, 31, 65, 64)])
def test_products_in_binary32(m, N, C, K, H, W):
    # edges of the 64 x 64 and 64 x 32 tiles, channel loops that end inside a group of eight channels
    print(f"[case] binary32 products F({m},3) N={N} C={C} K={K} {H}x{W}", flush=True)
    t = nova.nova_make_transforms(synth.point_set("standard" if m == 2 else "nova", m), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(C + K)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen)
    U = nova.nova_filter_transform(t, torch.randn((K, C, 3, 3), device=DEV, generator=gen) * (2.0 / (9 * C)) ** 0.5)
    n2, T = t.n * t.n, N * -(-H // m) * -(-W // m)
    V = nova.nova_input_transform(t, x)
    M = unblock(nova.nova_contract(t, U, V, N, C, H, W, K), n2, -(-T // 128) * 128, K)[:, :T].double()
    Ul, Vl = unblock(U, n2, -(-K // 32) * 32, C)[:, :K].double(), unblock(V, n2, T, C).double()
    want = torch.matmul(Vl, Ul.transpose(1, 2).contiguous())
    size = torch.matmul(Vl.abs(), Ul.abs().transpose(1, 2).contiguous())
    # C products, each rounded or not, and C sums in binary32; twice the standard bound as above
    assert ((M - want).abs() <= 2 * (2 * C + 2) * 2.0 ** -24 * size + 1e-37).all()


def block(a, rows):
    # [n2][t or k][C] -> the flat blocked layout [n2][C/32][rows][32], zero padded
    n2, have, C = a.shape
    out = torch.zeros((n2, rows, -(-C // 32) * 32), dtype=a.dtype, device=a.device)
    out[:, :have, :C] = a
    return out.view(n2, rows, -1, 32).transpose(1, 2).contiguous().view(-1)


@pytest.mark.parametrize("dtype,scale_v,scale_u", [(torch.float32, 2.0 ** -70, 2.0 ** -68),        # the products are subnormal
                                                   (torch.float32, 2.0 ** -130, 1.0), (torch.float32, 1.0, 2.0 ** -135),
                                                   (torch.float16, 2.0 ** -18, 1.0), (torch.float16, 1.0, 2.0 ** -20)])
@pytest.mark.parametrize("C,K", [(5, 20), (70, 65)])
def test_subnormal_operands_and_products(dtype, scale_v, scale_u, C, K):
    # operands handed to the contraction directly: nothing may be flushed to zero
    print(f"[case] subnormal products {dtype} V {scale_v} U {scale_u} C={C} K={K}", flush=True)
    m, N, H, W = 2, 1, 20, 23
    t = nova.nova_make_transforms(synth.point_set("standard", 2), 2, 3)
    n2, T = t.n * t.n, N * -(-H // m) * -(-W // m)
    gen = torch.Generator(device=DEV).manual_seed(C)
    V = (torch.randint(1, 64, (n2, T, C), device=DEV, generator=gen).double() * scale_v).to(dtype)
    U = (torch.randint(-63, 64, (n2, K, C), device=DEV, generator=gen).double() * scale_u).to(dtype)
    assert (V.double() / scale_v).abs().max() < 64 and (V.double() == (V.double() / scale_v).round() * scale_v).all()
    M = nova.nova_contract(t, block(U, -(-K // 32) * 32), block(V, T), N, C, H, W, K)
    M = unblock(M, n2, -(-T // 128) * 128, K)[:, :T].double()
    # whole multiples of scale_v * scale_u below 2^24 of them: every product and partial sum is exact
    assert torch.equal(M, torch.matmul(V.double(), U.double().transpose(1, 2).contiguous()))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("C,K,H", [(5, 20, 20), (70, 65, 20), (64, 128, 20)])
def test_operands_that_are_not_finite(dtype, C, K, H):
    # an infinity or NaN reaches the products of its own row and column and no others
    print(f"[case] contraction of values that are not finite {dtype} C={C} K={K}", flush=True)
    t = nova.nova_make_transforms(synth.point_set("standard", 2), 2, 3)
    n2, T = t.n * t.n, (H // 2) ** 2
    gen = torch.Generator(device=DEV).manual_seed(C)
    V, U = (torch.randint(-9, 10, (n2, rows, C), device=DEV, generator=gen).to(dtype) for rows in (T, K))
    V[1, 3, 2], V[1, 7, C - 1], V[2, T - 1, 0], V[3, 0, 1] = float("inf"), float("-inf"), float("nan"), float("inf")
    U[2, K - 1, C - 1], U[3, 4, 0], U[4, 0, 3], U[3, 5, 1] = float("inf"), float("nan"), float("-inf"), float("-inf")
    U[1, 6, 2] = 0.0                                                       # infinity times zero
    M = nova.nova_contract(t, block(U, -(-K // 32) * 32), block(V, T), 1, C, H, H, K)
    M = unblock(M, n2, -(-T // 128) * 128, K)[:, :T].double()
    want = torch.zeros((n2, T, K), dtype=torch.float64, device=DEV)
    for c in range(C):
        want += V[:, :, c, None].double() * U[:, None, :, c].double()      # (integers: the finite sums are exact)
    assert want.isinf().any() and want.isnan().any() and want.isfinite().any()
    assert torch.equal(M.isnan(), want.isnan()) and torch.equal(M.nan_to_num(nan=0.0), want.nan_to_num(nan=0.0))
