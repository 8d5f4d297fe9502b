"""What the header says of a served image's bits: those of gs_render_fwd_seg for the
selected Gaussians alone where that composites in the server's segments of 512
positions (4097 to 12288 tiles), and of gs_render_fwd with persistent compositing
at any size; batched with a small image or not."""
import math

import numpy as np
import pytest
import torch

import synthetic as S
import test_gpu_serving as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("persistent", [0, 64])
def test_bits_of_a_served_image(gpu_lib, persistent):
    gs, n = gpu_lib, 6000
    rng = np.random.default_rng(3)
    sc = S.random_scene(n, seed=6, log_scale_mu=-1.5)
    sc.means[:] = (0.3 * sc.means).astype(np.float32)
    sc.opacities[:] = rng.uniform(0.005, 0.02, n).astype(np.float32)
    params = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in sc.param_arrays()]
    table = gs.LodTable(np.full((1, 3), -9.0, np.float32), np.full((1, 3), 9.0, np.float32), np.zeros((3, 1), np.int64),
                        np.full((3, 1), n), (12.0, 24.0, math.inf), 0.1)
    opts = gs.RenderOptions(sh_degree=3, aa=True)
    cams = [S.Camera(1.2 * W, 1.2 * W, W / 2.0, H / 2.0, S.look_at((0.5, 0.2, -6.0), (0, 0, 0), up=(0, -1, 0)), W, H)
            for W, H in ((1040, 1024), (1600, 1072), (96, 64))]
    cfg = gs.ServeConfig(max_views_per_batch=3, n_streams=1, slot_capacity=4 * n, pair_capacity=20_000_000,
                         pixel_capacity=1 << 22, persistent_ctas=persistent, pairs_per_gaussian=500.0)
    outs, done, _ = T.serve(gs, params, table, opts, [(c, 10 ** 9) for c in cams], cfg, t_arrival=1.0)
    assert all(d["status"] == 0 and d["batch_views"] == 3 for d in done)
    longest = 0
    for cam, out in zip(cams, outs):
        proj = gs.project(*params, [cam], opts)
        pairs, ranges, _ = gs.bin_sort(proj, [cam], n)
        longest = max(longest, int((ranges[:, 1] - ranges[:, 0]).max()))
        ref = gs.render_fwd(proj, pairs, ranges, [cam], opts, seg=False if persistent else None)["rgb"].view_as(out)
        if persistent or 4096 < ranges.shape[0] <= 12288:
            assert torch.equal(out, ref)
        else:
            assert float((out - ref).abs().max()) <= 2e-5
    assert longest > 1024      # lists past the head
