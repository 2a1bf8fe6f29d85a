"""V = B^T d B at the edges of the input transform's work groups, bit for bit against the CPU oracle.

A workgroup takes 4, 8 or 16 consecutive tiles of the batch and the columns a window shares with its
neighbours come from the lanes beside it, except at the ends of a group: tile counts one below, at and one
above a group, groups that straddle tile rows and images, the last elements of x, odd channel counts and
values of x that start at any element.
"""
from fractions import Fraction as Fr

import numpy as np
import pytest
import torch

from oracle import conv
from paper_2512_18453_amd import nova, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # m, r, N, C, H, W
    (8, 3, 1, 2, 8, 56), (8, 3, 1, 1, 8, 64), (8, 3, 1, 33, 8, 65),        # 7, 8 and 9 tiles in one row
    (8, 3, 3, 5, 17, 19), (8, 3, 9, 3, 7, 7), (8, 3, 2, 31, 16, 121),      # rows and images inside a group; 16 columns + 1
    (6, 3, 1, 34, 13, 97), (6, 3, 17, 1, 6, 6), (6, 3, 2, 7, 11, 50),
    (4, 3, 1, 35, 4, 61), (4, 3, 1, 1, 5, 64), (4, 3, 18, 2, 3, 4),        # 16 tiles per group
    (2, 3, 2, 3, 7, 33), (2, 3, 1, 65, 2, 2),
    (2, 5, 1, 3, 6, 31), (2, 5, 5, 2, 3, 3),                               # two halo columns of two-column tiles
    (4, 5, 1, 5, 9, 33), (6, 5, 3, 9, 13, 49), (6, 5, 2, 33, 7, 6),
]


def tiles_of(V, n2, T, C):
    return V.cpu().numpy().reshape(n2, -(-C // 32), T, 32).transpose(0, 2, 1, 3).reshape(n2, T, -1)


@pytest.mark.parametrize("m,r,N,C,H,W", CASES)
@pytest.mark.parametrize("symmetric", [True, False])
def test_group_edges_bit_for_bit(m, r, N, C, H, W, symmetric):
    size = m + r - 3
    points = synth.point_set("standard" if size == 2 else "nova", size)
    if not symmetric:
        points = points[1:] + points[:1]                                   # the general kernels
    t = nova.nova_make_transforms(points, m, r)
    assert t.symmetric == symmetric
    rng = np.random.default_rng(100 * m + W)
    T = N * -(-H // m) * -(-W // m)
    for dtype, storage in ((np.float16, 16), (np.float32, 32)):
        print(f"[case] input transform F({m},{r}) {np.dtype(dtype).name} N={N} C={C} H={H} W={W} paired={symmetric}", flush=True)
        x = rng.standard_normal((N, C, H, W)).astype(dtype)
        w = np.zeros((1, C, r, r), dtype)
        _, _, want, _ = conv.winograd_conv2d_emulated(x.astype(np.float64), w.astype(np.float64), [Fr(a, b) for a, b in points], m,
                                                      storage=storage, want_intermediates=True)
        for shift in (0, 1, 3):                                            # x at any element of a larger buffer, NaN around it
            room = torch.full((x.size + shift,), float("nan"), dtype=torch.from_numpy(x).dtype, device=DEV)
            room[shift:] = torch.from_numpy(x.ravel()).to(DEV)
            V = nova.nova_input_transform(t, room[shift:].view(N, C, H, W))
            got = tiles_of(V, t.n * t.n, T, C)
            assert not got[:, :, C:].any()                                 # padding channels
            assert np.array_equal(got[:, :, :C].astype(np.float64), want), (dtype, shift)


@pytest.mark.parametrize("m,r,N,C,H,W", [(8, 3, 1, 3, 8, 250), (8, 3, 1, 1, 8, 136), (8, 3, 2, 4, 9, 264), (6, 3, 1, 2, 6, 97),
                                         (4, 3, 3, 3, 5, 61), (4, 5, 1, 1, 4, 130), (6, 5, 9, 3, 7, 11), (2, 3, 1, 3, 2, 65)])
def test_compact_layout_of_few_channels(m, r, N, C, H, W):
    # with at most four channels the single call keeps V as [position][tile][4], at the start of its workspace:
    # runs of 16 tiles whose lanes exchange columns, groups of 16 and 32
    size = m + r - 3
    points = synth.point_set("standard" if size == 2 else "nova", size)
    t = nova.nova_make_transforms(points, m, r)
    rng = np.random.default_rng(m + W)
    T = N * -(-H // m) * -(-W // m)
    for dtype, storage in ((np.float16, 16), (np.float32, 32)):
        print(f"[case] compact input transform F({m},{r}) {np.dtype(dtype).name} N={N} C={C} H={H} W={W}", flush=True)
        x = rng.standard_normal((N, C, H, W)).astype(dtype)
        _, _, want, _ = conv.winograd_conv2d_emulated(x.astype(np.float64), np.zeros((1, C, r, r)), [Fr(a, b) for a, b in points], m,
                                                      storage=storage, want_intermediates=True)
        dt = nova.NOVA_F16 if storage == 16 else nova.NOVA_F32
        ws = torch.zeros(nova.nova_conv2d_workspace_bytes(N, C, H, W, 5, m, dt, 0, N, r), dtype=torch.uint8, device=DEV)
        U = torch.zeros(nova.nova_filter_bytes(5, C, m, dt, r) // (storage // 8), dtype=torch.from_numpy(x).dtype, device=DEV)
        nova.nova_winograd_conv2d(t, torch.from_numpy(x).to(DEV), U, 5, workspace=ws)
        Vc = ws.view(U.dtype)[:t.n * t.n * T * 4].cpu().numpy().reshape(t.n * t.n, T, 4).astype(np.float64)
        assert np.array_equal(Vc[:, :, :C], want) and not Vc[:, :, C:].any()


@pytest.mark.parametrize("m,r", [(2, 3), (4, 3), (6, 3), (8, 3), (2, 5), (4, 5), (6, 5)])
def test_large_launches_equal_small_ones(m, r):
    # launches of no more workgroups than compute units share a tile among more threads: the whole batch
    # (several times as many workgroups) against single images, bit for bit
    size = m + r - 3
    t = nova.nova_make_transforms(synth.point_set("standard" if size == 2 else "nova", size), m, r)
    gen = torch.Generator(device=DEV).manual_seed(m + r)
    N, C, H, W = 24, 70, 9 * m + 1, 11 * m - 1
    per, n2 = -(-H // m) * -(-W // m), t.n * t.n
    for dtype in (torch.float16, torch.float32):
        print(f"[case] large and small launches F({m},{r}) {dtype}", flush=True)
        x = torch.randn((N, C, H, W), device=DEV, generator=gen).to(dtype)
        V = nova.nova_input_transform(t, x).view(n2, 3, N, per, 32)
        for i in (0, 7, N - 1):
            assert torch.equal(V[:, :, i], nova.nova_input_transform(t, x[i:i + 1].contiguous()).view(n2, 3, per, 32))


def test_streamed_input_gives_the_same_result():
    # x, V and M together larger than the last-level cache and one tile row per group: the whole batch in one
    # pass against slabs that fit
    N, C, K, H, W, m = 40, 256, 256, 56, 56, 8
    print(f"[case] streamed x, F({m},3) fp16 N={N} C={C} K={K} {H}x{W}", flush=True)
    t = nova.nova_make_transforms(synth.point_set("nova", m), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((N, C, H, W), device=DEV, generator=gen).half()
    U = nova.nova_filter_transform(t, (torch.randn((K, C, 3, 3), device=DEV, generator=gen) * 0.03).half())
    whole = nova.nova_winograd_conv2d(t, x, U, K, images_per_slab=N)
    slabs = nova.nova_winograd_conv2d(t, x, U, K, images_per_slab=4)
    assert torch.isfinite(whole).all() and torch.equal(whole, slabs)


def test_planes_beyond_32_bit_offsets():
    # 32 channel planes of 2^30 elements: addresses are formed element by element; the tiles of the first
    # columns against the same columns as an image of their own
    m, H, W = 8, 512, 65536
    print(f"[case] input transform F({m},3) fp16 {H}x{W}", flush=True)
    t = nova.nova_make_transforms(synth.point_set("nova", m), m, 3)
    gen = torch.Generator(device=DEV).manual_seed(6)
    x = torch.randn((1, 1, H, W), device=DEV, generator=gen).half()
    V = nova.nova_input_transform(t, x).view(t.n * t.n, 1, H // m, W // m, 32)
    part = nova.nova_input_transform(t, x[:, :, :, :64].contiguous()).view(t.n * t.n, 1, H // m, 8, 32)
    assert torch.equal(V[:, :, :, :7], part[:, :, :, :7])                  # (the eighth tile's right halo differs)
    last = nova.nova_input_transform(t, x[:, :, :, -64:].contiguous()).view(t.n * t.n, 1, H // m, 8, 32)
    assert torch.equal(V[:, :, :, -7:], last[:, :, :, -7:])
