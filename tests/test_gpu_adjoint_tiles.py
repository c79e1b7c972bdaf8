"""Adjoint tiles at their edges: frames one row or column short of, equal to
and past a tile, for every tile shape, under motion that mixes rigid, random
and converging parts (many pixels onto one cell), against the float64 oracle."""

import numpy as np
import pytest
import torch

import paper_2307_12607_amd as exw
from oracle import warp_oracle
from gpu_util import announce, half_ulp, need_gpu, stored, to_dev, to_host

pytestmark = pytest.mark.gpu

# (channels, phases, tile rows): one entry per tile shape of the kernel
SHAPES = [(1, 1, 32), (2, 3, 16), (3, 1, 16), (3, 3, 16), (4, 3, 12), (4, 4, 12), (12, 1, 4),
          (12, 1, 6), (12, 2, 6), (12, 3, 4), (12, 4, 6)]
PHASES = [0.25, 0.5, 0.75, 1.0]


def mixed_motion(rng, h, w):
    """Rigid top, random middle, bottom rows that all sample one pixel."""
    mv = np.empty((1, 2, h, w), np.float32)
    mv[:, 0], mv[:, 1] = 2.75, -1.5
    a, b = h // 3, 2 * h // 3
    mv[:, :, a:b] = rng.uniform(-5, 5, size=(1, 2, b - a, w))
    x = np.arange(w, dtype=np.float32)
    mv[:, 0, b:] = x - np.float32(min(w - 1, 70) - 0.375)
    mv[:, 1, b:] = 0.25
    return mv


@pytest.mark.parametrize("c,k,rows", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tile_edges(c, k, rows, dtype):
    dev = need_gpu()
    phases = [1.0] if k == 1 else PHASES[:k]
    rng = np.random.default_rng(100 * c + k)
    for h, w in ((rows - 1, 127), (rows, 128), (rows + 1, 129), (2 * rows + 1, 191), (3, 2),
                 (5, 1)):
        announce("tiles", c, k, h, w, dtype)
        src = rng.random((1, c, h, w), dtype=np.float32)
        mv = mixed_motion(rng, h, w)
        g = rng.standard_normal((1, k, c, h, w)).astype(np.float32)
        src_q, g_q = stored(src, dtype), stored(g, dtype)
        ref_gs, ref_gm = warp_oracle.backward(src_q, mv, phases, g_q)
        # sums of |weight * g|, and of the motion gradient's terms: float32
        # products round by 2^-24 each, a few per term, so 2^-19 of the sum of
        # magnitudes (at least of 1) bounds them
        abs_gs, _ = warp_oracle.backward(src_q, mv, phases, np.abs(g_q))
        abs_gm = np.abs(g_q).sum(axis=(1, 2))[:, None]
        gs, gm = exw.warp_backward(to_dev(src, dtype, dev), torch.from_numpy(mv).to(dev), phases,
                                   to_dev(g, dtype, dev))
        torch.cuda.synchronize()
        tol = 2.0 ** -19
        bound = tol * np.maximum(1.0, abs_gs)
        if dtype != "f32":
            bound = bound + half_ulp(ref_gs, dtype)
        assert (np.abs(to_host(gs) - ref_gs) <= bound).all(), (h, w)
        assert (np.abs(to_host(gm) - ref_gm) <= tol * np.maximum(1.0, abs_gm)).all(), (h, w)


def test_more_frames_than_one_launch_of_tiles_holds():
    """2^23 + 3 frames of one pixel: the tiles take two launches. Motion 0, so
    the image gradient is the upstream gradient."""
    dev = need_gpu()
    n = (1 << 23) + 3
    announce("tiny frames", n)
    g = torch.arange(n, device=dev, dtype=torch.float32).view(n, 1, 1, 1, 1) - 0.5
    gs, _ = exw.warp_backward(torch.ones(n, 1, 1, 1, device=dev), torch.zeros(n, 2, 1, 1, device=dev),
                              [1.0], g)
    torch.cuda.synchronize()
    assert torch.equal(gs, g[:, 0])


@pytest.mark.parametrize("c", [1, 2, 3, 4, 12])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_sums_are_float64_and_rounded_at_the_end(c, dtype):
    """Motion in eighths and whole upstream gradients: every weight, product
    and float64 sum is exact, whatever the order of the additions, also where
    hundreds of pixels meet in one cell (where float32 sums would round). The
    image gradient is then the exact sum rounded to float32 and to the storage
    type, in every run. (The segments from column 256 on of the converging rows
    lie more than 128 pixels from that cell: their contributions are float32
    atomics, and the cells they reach are only bounded.)"""
    dev = need_gpu()
    rng = np.random.default_rng(c)
    h, w, phases = 40, 300, [0.5, 1.0]
    mv = mixed_motion(rng, h, w)
    mv[:, :, h // 3:2 * h // 3] = rng.integers(-40, 41, mv[:, :, h // 3:2 * h // 3].shape) / 8
    # storable in every type: 8 significant bits
    g = (rng.integers(-255, 256, (1, 2, c, h, w)) * 4096.0 + 0.0).astype(np.float32)
    g[:, :, :, ::2] /= 4096.0
    if dtype == "f16":
        g /= 64.0  # within its range
    src = rng.random((1, c, h, w), dtype=np.float32)
    exact, _ = warp_oracle.backward(src, mv, phases, g)
    want = torch.from_numpy(exact).to(torch.float32).to({"f32": torch.float32, "f16": torch.float16,
                                                         "bf16": torch.bfloat16}[dtype])
    far = np.zeros_like(g)
    far[..., 2 * (h // 3):, 256:] = 1.0
    by_atomics = torch.from_numpy(warp_oracle.backward(src, mv, phases, far)[0] != 0)
    # at most 512 additions to a cell, each rounding by 2^-24 of the magnitudes
    bound = torch.from_numpy(2.0 ** -15 * warp_oracle.backward(src, mv, phases, np.abs(g))[0]
                             + (0.0 if dtype == "f32" else half_ulp(exact, dtype)))
    # (sums beyond float16's range are infinite)
    bounded = by_atomics & (torch.from_numpy(np.abs(exact)) + bound < torch.finfo(want.dtype).max)
    assert bounded.any() and by_atomics.float().mean() < 0.2
    announce("exact sums", c, dtype)
    args = (to_dev(src, dtype, dev), torch.from_numpy(mv).to(dev), phases, to_dev(g, dtype, dev))
    for _ in range(3):
        gs, _ = exw.warp_backward(*args)
        torch.cuda.synchronize()
        gs = gs.cpu()
        assert torch.equal(gs[~by_atomics], want[~by_atomics])
        err = (gs.double() - torch.from_numpy(exact)).abs()
        assert (err[bounded] <= bound[bounded]).all()
