"""The served projection's chunks of slots where their segments end: many
segments of one Gaussian in a chunk (each slot searches its own), a few, one
over many chunks, and enough slots for chunks of 256; several views a batch.

A request's image must be that of rendering the selected Gaussians directly:
same slots in the same order, composited with other segment lengths, so equal
to some float32 roundings of values of at most 1 (2e-5)."""
import math

import numpy as np
import pytest
import torch

import synthetic as S
import test_gpu_serving as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes", [(1, (1, 1)), (63, (1, 1)), (300, (1, 1)), (300, (1, 3)), (1000, (5, 40)), (5000, (5000, 5000)),
                                     (4097, (60, 70)), (620_000, (1, 8)), (620_000, (30, 400))])
def test_segment_sizes(gpu_lib, n, sizes):
    gs = gpu_lib
    rng = np.random.default_rng(n + sizes[0])
    sc = S.random_scene(n, seed=n % 1000, log_scale_mu=-4.0 if n > 10_000 else -2.0)
    arrays = [np.ascontiguousarray(a) for a in sc.param_arrays()]
    arrays[3] = (arrays[3] * (0.05 if n > 10_000 else 1.0)).astype(np.float32)
    counts = []
    while sum(counts) < n:
        counts.append(min(int(rng.integers(sizes[0], sizes[1] + 1)), n - sum(counts)))
    counts = np.asarray(counts, np.int64)
    parts = len(counts)
    offsets = np.concatenate([[0], np.cumsum(counts)[:-1]])
    lo, hi = np.full((parts, 3), -3.0, np.float32), np.full((parts, 3), 3.0, np.float32)
    # the same Gaussians at every level
    table = gs.LodTable(lo, hi, np.stack([offsets] * 3), np.stack([counts] * 3), (12.0, 24.0, math.inf), 0.1)
    params = [torch.from_numpy(a).cuda() for a in arrays]
    opts = gs.RenderOptions(sh_degree=3, aa=True)
    cams = []
    for k in range(3):
        W, H = ((40, 33), (64, 48), (31, 57))[k]
        eye = (0.7 * np.sin(2.0 * k), 0.2 * k, -4.0)
        cams.append(S.Camera(1.2 * W, 1.2 * W, W / 2.0, H / 2.0, S.look_at(eye, (0, 0, 0), up=(0, -1, 0)), W, H))
    cfg = gs.ServeConfig(max_views_per_batch=3, n_streams=1, slot_capacity=4 * max(n, 1000), pair_capacity=40_000_000,
                         pixel_capacity=1 << 20)
    outs, _, _ = T.serve(gs, params, table, opts, [(c, 10 ** 9) for c in cams], cfg)
    for cam, out in zip(cams, outs):
        rgb, _, _ = gs.rasterize(*params, [cam], opts)
        ref = rgb.detach().view(cam.height, cam.width, 3)
        assert float((out - ref).abs().max()) <= 2e-5
