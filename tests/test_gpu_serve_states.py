"""Served batches whose lists fill the pair buffer: the segment states of all their
views fit the server's area, so the batch is composited in segments and an image has
the same bits alone (where the states always fit) and in a full batch.

Every Gaussian covers a whole image of 80 tiles, so a tile's list holds all n = 16000
and leaves 31 states: 9920 for four views."""
import math

import numpy as np
import pytest
import torch

import synthetic as S
import test_gpu_serving as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pixel_capacity", [1 << 17, 1 << 18, 1 << 20])
def test_dense_batch_alone_and_together(gpu_lib, pixel_capacity):
    gs, n, W, H = gpu_lib, 16_000, 160, 128
    rng = np.random.default_rng(2)
    sc = S.random_scene(n, seed=1, log_scale_mu=3.6, log_scale_sigma=0.05)
    sc.means[:] = (0.05 * sc.means).astype(np.float32)
    sc.opacities[:] = rng.uniform(0.0042, 0.0044, n).astype(np.float32)
    params = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in sc.param_arrays()]
    lo, hi = np.full((1, 3), -9.0, np.float32), np.full((1, 3), 9.0, np.float32)
    table = gs.LodTable(lo, hi, np.zeros((3, 1), np.int64), np.full((3, 1), n), (12.0, 24.0, math.inf), 0.1)
    opts = gs.RenderOptions(sh_degree=3)
    cams = [S.Camera(60.0, 60.0, W / 2.0, H / 2.0, S.look_at((0.3 * k, 0.1, -6.0), (0, 0, 0), up=(0, -1, 0)), W, H)
            for k in range(4)]
    proj = gs.project(*params, cams, opts)
    P = int(proj.tiles.long().sum())
    tiles = 4 * (W // 16) * (H // 16)
    assert P >= 0.95 * n * tiles
    one = dict(n_streams=1, slot_capacity=4 * n, pixel_capacity=pixel_capacity, pairs_per_gaussian=0.9 * P / (4 * n))
    # room for the four views and not much more
    cfg = gs.ServeConfig(max_views_per_batch=4, pair_capacity=int(1.1 * P), **one)
    reqs = [(c, 10 ** 9) for c in cams]
    outs, done, _ = T.serve(gs, params, table, opts, reqs, cfg, t_arrival=1.0)      # all four have arrived
    assert all(d["status"] == 0 and d["batch_views"] == 4 for d in done)
    alone = gs.ServeConfig(max_views_per_batch=1, pair_capacity=int(1.1 * P), **one)
    for req, out in zip(reqs, outs):
        ref, _, _ = T.serve(gs, params, table, opts, [req], alone)
        assert float(out.abs().max()) > 0.0
        assert torch.equal(out, ref[0])
