"""nova_winograd_conv2d_int8 (maxima left by the input transform, V quantised inside the contraction) against the
stage calls (maxima, codes and contraction one by one), bit for bit: both take every deciding step in the
same correctly rounded binary32 arithmetic."""
import pytest
import torch

from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MODES = (nova.NOVA_INT8_PER_TENSOR, nova.NOVA_INT8_PER_CHANNEL, nova.NOVA_INT8_PER_POSITION)

CASES = [
    # m, N, C, K, H, W, dtype, points in the paired order
    (4, 1, 1, 1, 3, 3, torch.float16, True),              # one tile: the partial maxima do not fit, separate passes
    (4, 1, 33, 129, 4, 65, torch.float16, True),          # 17 tiles, one more channel than a block / a column block
    (6, 2, 31, 128, 42, 25, torch.float32, True),
    (8, 1, 40, 70, 57, 63, torch.float16, True),          # 64 tiles
    (2, 3, 64, 40, 17, 31, torch.float16, True),          # 128 * 3 tiles: whole row blocks
    (4, 2, 24, 40, 18, 20, torch.float16, False),         # general kernels: separate passes
    (4, 40, 64, 32, 130, 130, torch.float16, True),       # more partial maxima than a workgroup reads by itself
    (8, 12, 40, 33, 120, 120, torch.float32, True),
]


def both(t, x, w, mode, flags=0):
    N, C, H, W = x.shape
    K = w.shape[0]
    Uq, su = nova.nova_quantize_filter_int8(t, nova.nova_filter_transform(t, w), K, C, mode)
    Vq, sv = nova.nova_quantize_input_int8(t, nova.nova_input_transform(t, x), N, C, H, W, mode)
    M = nova.nova_contract_int8(t, Uq, Vq, su, sv, mode, N, C, H, W, K, dequantise=True)
    want = nova.nova_output_transform(t, M, N, K, H, W, x.dtype, flags)
    ws = torch.full((nova.nova_conv2d_int8_workspace_bytes(N, C, H, W, K, t.m, nova._dtype_code(x), t.r),), 0xFF, dtype=torch.uint8,
                    device=DEV)                                        # NaN everywhere
    return nova.nova_winograd_conv2d_int8(t, x, Uq, su, mode, K, flags=flags, workspace=ws), want, sv


@pytest.mark.parametrize("m,N,C,K,H,W,dtype,paired", CASES)
def test_single_call_equals_the_stages(m, N, C, K, H, W, dtype, paired):
    points = synth.point_set("standard" if m == 2 else "nova", m)
    t = nova.nova_make_transforms(points if paired else points[1:] + points[:1], m, 3)
    assert t.symmetric == paired
    gen = torch.Generator(device=DEV).manual_seed(m + W)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
    w = (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * (2.0 / (9 * C)) ** 0.5).to(dtype)
    for mode in MODES:
        print(f"[case] int8 single call F({m},3) {dtype} mode {mode} N={N} C={C} K={K} H={H} W={W}", flush=True)
        got, want, _ = both(t, x, w, mode)
        assert torch.isfinite(want).all() and torch.equal(got, want)


def test_ties_round_to_even_as_in_the_stages():
    # integer V with largest magnitude 254, hence s = 2: every odd value is a tie
    t = nova.nova_make_transforms(synth.point_set("standard", 2), 2, 3)
    gen = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randint(-60, 61, (2, 40, 22, 30), device=DEV, generator=gen).half()
    x[0, 3, 5:8, 7:10] = 0                           # one window (tile row 3, column 4): d00 - d02 - d20 + d22 = 254
    x[0, 3, 5, 7], x[0, 3, 5, 9], x[0, 3, 7, 7], x[0, 3, 7, 9] = 64, -63, -63, 64
    w = torch.randn((33, 40, 3, 3), device=DEV, generator=gen).half()
    got, want, sv = both(t, x, w, nova.NOVA_INT8_PER_TENSOR)
    assert sv.item() == 2.0 and torch.equal(got, want)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_values_that_are_not_finite(bad):
    t = nova.nova_make_transforms(synth.point_set("nova", 4), 4, 3)
    gen = torch.Generator(device=DEV).manual_seed(4)
    x = torch.randn((1, 8, 20, 20), device=DEV, generator=gen).half()
    x[0, 2, 9, 9] = bad
    w = torch.randn((16, 8, 3, 3), device=DEV, generator=gen).half()
    for mode in MODES:
        got, want, _ = both(t, x, w, mode)
        assert torch.equal(got.nan_to_num(nan=7.0), want.nan_to_num(nan=7.0))


# Tile counts that leave the last group of the input transform part empty, the image a whole number of tiles wide, so that
# the last tile's own last columns are not zero: what a lane without a tile reads must not reach the maxima.
# (m, r, last tile's own columns, the columns left of them): patterns for which a window whose left halo repeats the
# tile's own last columns would exceed every real one (no such pattern of 0 and +-1 exists for two-column tiles).
PATTERNS = [
    (4, 3, (0, 0, 0, -1), (0,)),
    (6, 3, (-1, -1, -1, 0, -1, 1), (-1,)),
    (8, 3, (-1, 0, -1, -1, -1, -1, -1, -1), (1,)),
    (4, 5, (-1, -1, 0, 0), (-1, -1)),
    (6, 5, (-1, -1, -1, 0, 0, 1), (-1, -1)),
]


@pytest.mark.parametrize("m,r,own,left", PATTERNS)
@pytest.mark.parametrize("N,tiles", [(1, 3), (1, 5), (3, 3)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_lanes_without_a_tile_leave_the_scale_alone(m, r, own, left, N, tiles, dtype):
    t = nova.nova_make_transforms(synth.point_set("nova", m + r - 3), m, r)
    C, K, H, W = 35, 33, tiles * m, tiles * m
    pad = (r - 1) // 2
    gen = torch.Generator(device=DEV).manual_seed(m + r + tiles)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen) * 0.01
    cols = torch.tensor(left + own, dtype=torch.float32, device=DEV)
    x[-1, 34, H - m - pad:, W - m - pad:] = cols[:, None] * cols * 4
    B = torch.tensor(nova.nova_get_matrix_f64(t, nova.NOVA_MATRIX_BT), dtype=torch.float64)
    repeated = torch.nn.functional.pad(x[-1, 34, H - m - pad:, W - m - pad:].cpu().double(), (0, pad, 0, pad))
    repeated[:, :pad] = repeated[:, m:m + pad].clone()
    beyond = (B @ repeated @ B.t()).abs().max().item()
    w = (torch.randn((K, C, r, r), device=DEV, generator=gen) * 0.1).to(dtype)
    for mode in MODES:
        print(f"[case] int8 planted maximum F({m},{r}) {dtype} mode {mode} N={N} {H}x{W}", flush=True)
        got, want, sv = both(t, x.to(dtype), w, mode)
        assert sv.max().item() * 127 * 1.05 < beyond              # (the pattern does what it is there for)
        assert torch.isfinite(want).all() and torch.equal(got, want)


@pytest.mark.parametrize("m,N,C,K,H,W", [(4, 1, 64, 32, 12, 12), (4, 1, 16, 33, 20, 20), (4, 1, 64, 64, 28, 28), (2, 1, 40, 32, 10, 10),
                                         (6, 1, 64, 32, 18, 18), (6, 3, 33, 40, 30, 24), (8, 3, 64, 32, 24, 24), (8, 1, 40, 70, 40, 40)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_ragged_groups_of_whole_tiles(m, N, C, K, H, W, dtype):
    t = nova.nova_make_transforms(synth.point_set("standard" if m == 2 else "nova", m), m, 3)
    for seed in range(6):
        gen = torch.Generator(device=DEV).manual_seed(seed)
        x = torch.randn((N, C, H, W), device=DEV, generator=gen).abs().to(dtype)
        w = (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * (2.0 / (9 * C)) ** 0.5).to(dtype)
        for mode in MODES:
            print(f"[case] int8 ragged groups F({m},3) {dtype} mode {mode} N={N} C={C} K={K} {H}x{W} seed {seed}", flush=True)
            got, want, _ = both(t, x, w, mode)
            assert torch.isfinite(want).all() and torch.equal(got, want)
