"""Rows of tiles that the right edge cuts off leave in pieces of 4, 2 and 1 values: every number of columns that a last tile can keep, from each
kernel that stores rows, straight from registers (three tiles and the last) and through LDS (one tile, two tiles).  Against the same call on
the image with zeros appended up to whole tiles, whose rows are all whole: the same windows, hence the same bits."""
import pytest
import torch

from launches import launches
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F16, F32 = torch.float16, torch.float32

# kernel that leaves the results, m, r, C, K, images at one tile each
CASES = [("contract_output_kernel", m, r, C, 70, n) for m, r, C, n in ((2, 3, 100, 16000), (4, 3, 160, 9000), (6, 3, 100, 8000), (2, 5, 100, 8000), (4, 5, 100, 8000), (6, 5, 100, 15000))]
CASES += [("fused_contract_output_kernel", 6, 3, 64, 64, 30000), ("fused_contract_output_kernel", 8, 3, 64, 64, 30000)]
CASES += [("few_channels_kernel", m, r, 3, 40, 300) for m, r in ((2, 3), (4, 3), (6, 3), (8, 3), (2, 5), (4, 5), (6, 5))]
CASES += [("layer_kernel", m, r, 16, 33, 24) for m, r in ((2, 3), (4, 3), (6, 3), (8, 3), (2, 5), (4, 5), (6, 5))]
CASES += [("output_transform_kernel", m, r, 300, 128, 600) for m, r in ((4, 3), (6, 3), (8, 3))]


@pytest.mark.parametrize("kernel,m,r,C,K,images", CASES)
def test_every_number_of_columns(kernel, m, r, C, K, images):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m + C)
    w = torch.randn((K, C, r, r), device=DEV, generator=gen) * (2.0 / (r * r * C)) ** 0.5
    for dtype in (F16, F32) if kernel in ("layer_kernel", "output_transform_kernel") else (F16,):
        U = nova.nova_filter_transform(t, w.to(dtype))
        for tiles in (1, 2, 4):
            for left in range(1, m):
                W = (tiles - 1) * m + left
                N, H = -(-images // tiles), max(m - 1, 2)
                print(f"[case] {kernel} F({m},{r}) {dtype} N={N} C={C} K={K} {H}x{W}", flush=True)
                x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
                whole = torch.nn.functional.pad(x, (0, m - left))
                results = []
                for image in (x, whole):
                    y = torch.full((N, K, H, image.shape[3]), 7.0, dtype=dtype, device=DEV)
                    ws = torch.empty(nova.nova_conv2d_workspace_bytes(N, C, H, image.shape[3], K, m, nova.NOVA_F16 if dtype == F16 else nova.NOVA_F32, 0, 0, r),
                                     dtype=torch.uint8, device=DEV)
                    nova.nova_winograd_conv2d(t, image, U, K, y=y, workspace=ws)
                    if image is x:
                        last = launches(lambda: nova.nova_winograd_conv2d(t, x, U, K, y=y, workspace=ws))[-1][0]
                        assert last.startswith(kernel + "<"), last
                    results.append(y)
                torch.cuda.synchronize()
                assert torch.isfinite(results[0]).all() and torch.equal(results[0], results[1][..., :W])
