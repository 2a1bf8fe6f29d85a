"""Input transforms of few tiles take workgroups of four: tile counts around a group and around the last launch that does, odd channel
counts, against the same tiles in a launch many times as large, bit for bit (which the oracle confirms elsewhere)."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("m,r", [(4, 3), (6, 3), (8, 3), (2, 5), (4, 5), (6, 5)])
def test_small_launches(m, r):
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device=DEV).manual_seed(10 * m + r)
    C, H, W, n2 = 67, m - 1, 2 * m - 1, t.n * t.n                          # two tiles an image, three channel blocks
    for dtype in (torch.float16, torch.float32):
        edge = 4 * units * (2 if t.n == 6 and dtype == torch.float16 else 1) // 3 // 2
        N = 12 * units
        x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
        V = nova.nova_input_transform(t, x).view(n2, 3, N, 2, 32)
        for images in (1, 2, 3, edge - 1, edge, edge + 1, 2 * edge):
            print(f"[case] {images} images F({m},{r}) {dtype}", flush=True)
            part = nova.nova_input_transform(t, x[N - images:].contiguous()).view(n2, 3, images, 2, 32)
            assert torch.equal(part, V[:, :, N - images:])
