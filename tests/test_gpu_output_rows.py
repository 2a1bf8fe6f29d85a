"""How results leave where W is no whole number of 16-byte pieces: every number of columns that a last tile can keep, several images to a
workgroup with the last workgroup short of some, channels that end inside a block, y at any element -- against A^T M A
evaluated in binary64 on the M the kernel was given, with what lies around y untouched."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# m, r, then (N, K, H, W): last tiles of 1 .. m - 1 columns; one, two and four tiles per image; two groups per row
CASES = [(m, r, shape) for m, r in ((2, 3), (4, 3), (6, 3), (8, 3), (2, 5), (4, 5), (6, 5))
         for shape in [(3, 33, m + 1, 2 * m + rest) for rest in range(1, m)] + [(9, 5, m - 1, m - 1), (7, 40, m, m + 1), (5, 3, 2 * m - 1, 2 * m - 1),
                                                                               (2, 33, 3, 16 * m + 1)]]

# binary32 whose rows of a channel leave as one run (2) or piece by piece (0): M and y of 64 MB or more by the columns in the last tile, of 192, images of one
# tile with few rows and with more, a channel block that is not full
RUNS = [(4, 3, (60, 100, 43, 42), 2), (4, 3, (60, 100, 43, 41), 0), (4, 3, (58, 96, 30, 31), 2), (6, 3, (48, 64, 50, 50), 2), (6, 3, (20, 64, 50, 50), 0), (6, 5, (80, 65, 26, 26), 2),
        (8, 3, (512, 64, 15, 15), 2), (8, 3, (512, 64, 15, 13), 0), (6, 3, (40, 33, 3, 5), 2), (6, 3, (40, 33, 4, 5), 0), (8, 3, (40, 33, 4, 7), 2), (8, 3, (9, 40, 5, 7), 0),
        (6, 5, (9, 5, 2, 3), 2), (2, 3, (9, 5, 2, 3), 0), (2, 3, (70, 160, 30, 31), 2), (4, 3, (92, 96, 41, 41), 2), (4, 5, (70, 96, 39, 39), 2)]
CASES += [(m, r, shape) for m, r, shape, way in RUNS if way == 2]


@pytest.mark.parametrize("m,r,shape,way", RUNS)
def test_way_of_binary32(m, r, shape, way):
    N, K, H, W = shape
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    M = torch.zeros(nova.nova_product_bytes(N, K, H, W, m, nova.NOVA_F32, 0, r) // 4, device=DEV)
    around = torch.empty(N * K * H * W + 4, device=DEV)
    for shift in (0, 1):
        y = around[shift:shift + N * K * H * W].view(N, K, H, W)
        name = launches(lambda: nova.nova_output_transform(t, M, N, K, H, W, torch.float32, 0, y=y))[0][0]
        assert name.startswith(f"output_transform_kernel<{t.n}, {r}, float, float, 1, {0 if shift else way},"), name


@pytest.mark.parametrize("m,r,shape", CASES)
def test_rows_of_any_width(m, r, shape):
    N, K, H, W = shape
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    n, th, tw, kb = t.n, -(-H // m), -(-W // m), -(-K // 32)
    T = N * th * tw
    A = torch.tensor(nova.nova_get_matrix_f32(t, nova.NOVA_MATRIX_A), dtype=torch.float64, device=DEV)
    M = torch.randn((n * n, kb, -(-T // 128) * 128, 32), device=DEV, generator=torch.Generator(device=DEV).manual_seed(W + N))
    P = M[:, :, :T].double().permute(0, 2, 1, 3).reshape(n, n, T, kb * 32)[:, :, :, :K]

    def through(a, p):
        z = torch.tensordot(a, torch.tensordot(a, p, dims=([0], [0])), dims=([0], [1]))             # [q, p, T, K]
        return z.reshape(m, m, N, th, tw, K).permute(2, 5, 3, 1, 4, 0).reshape(N, K, th * m, tw * m)[:, :, :H, :W]

    want, size_of = through(A, P), through(A.abs(), P.abs())
    for dtype in (torch.float16, torch.float32):
        print(f"[case] rows F({m},{r}) {dtype} N={N} K={K} {H}x{W}", flush=True)
        # 2 n roundings of binary32 at most of the absolute sum, then one to the storage format
        bound = 2 * (2 * n + 2) * 2.0 ** -24 * size_of + (2.0 ** -11 * want.abs() + 2.0 ** -25 if dtype == torch.float16 else 0.0)
        for shift in (0, 1, 3):
            around = torch.full((N * K * H * W + 16,), 7.0, dtype=dtype, device=DEV)
            got = around[shift:shift + N * K * H * W].view(N, K, H, W)
            nova.nova_output_transform(t, M.reshape(-1), N, K, H, W, dtype, 0, y=got)
            assert ((got.double() - want).abs() <= bound).all(), float(((got.double() - want).abs() / bound).max())
            assert (around[:shift] == 7.0).all() and (around[shift + N * K * H * W:] == 7.0).all()
