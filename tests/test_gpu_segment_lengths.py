"""Segmented compositing in launches of each segment length (128, 512, 1024 and
2048 positions, by the launch's tiles), around the length itself, the head and
several segments: against the same lists walked whole, forward and backward.

Segments multiply their transmittances and add their sums in another order: a few
roundings of values of at most 1 in the forward (2e-6 per image value, 1e-5 for
depths to 5); in the backward the whole walk divides T back through thousands of
entries (one unit roundoff each at worst, in quadrature 5000^0.5 x 6e-8 = 4e-6
relative, times the cancellation in g.c - S): 2e-4 of each field's norm."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n", [(320, 200, 129), (320, 200, 3000), (1600, 1072, 513), (1600, 1072, 3000),
                                   (2112, 2000, 1024), (2112, 2000, 1025), (2112, 2000, 5000), (3008, 3000, 2048),
                                   (3008, 3000, 2049), (3008, 3000, 4097), (3008, 3000, 7000)])
def test_against_whole_lists(gpu_lib, W, H, n):
    rng = np.random.default_rng(n + W)
    scene = S.random_scene(n, seed=n, log_scale_mu=-1.0, log_scale_sigma=0.2)
    scene.means[:] = rng.uniform(-0.02, 0.02, scene.means.shape).astype(np.float32)
    scene.opacities[:] = rng.uniform(0.0045, 0.012, n).astype(np.float32)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(60.0, 60.0, W / 2.0 + 1.3, H / 2.0 - 2.1, vm, W, H)
    opts = gpu_lib.RenderOptions(aa=False, bg=(0.1, 0.4, 0.7))
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, _ = gpu_lib.bin_sort(proj, [cam], n)
    longest = int((ranges[:, 1] - ranges[:, 0]).max())
    assert longest >= n * 3 // 4
    seg = gpu_lib.seg_workspace([cam], pairs)
    none = torch.empty(256, dtype=torch.uint8, device="cuda")
    got = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=seg)
    ref = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=False)
    for k, tol in (("rgb", 2e-6), ("alpha", 2e-6), ("T", 2e-6), ("depth", 1e-5)):
        assert float((got[k] - ref[k]).abs().max()) <= tol, k
    # (a pixel whose T ends within rounding of the stop threshold may stop an entry apart)
    assert int((got["last"] != ref["last"]).sum()) <= 3
    same = got["last"] == ref["last"]
    g = [torch.from_numpy(rng.standard_normal((W * H, 3)).astype(np.float32)).cuda() * same[:, None],
         torch.from_numpy((0.2 * rng.standard_normal(W * H)).astype(np.float32)).cuda() * same,
         torch.from_numpy(rng.standard_normal(W * H).astype(np.float32)).cuda() * same]
    a = gpu_lib.grad2d_view(gpu_lib.render_bwd(params, [cam], opts, proj, pairs, ranges, got["T"], got["last"], *g,
                                               seg=seg)).clone()
    b = gpu_lib.grad2d_view(gpu_lib.render_bwd(params, [cam], opts, proj, pairs, ranges, ref["T"], ref["last"], *g,
                                               seg=none))
    seen = proj.tiles > 0
    for f in range(10):
        x, y = a[seen][:, f].double(), b[seen][:, f].double()
        assert float((x - y).norm()) <= 2e-4 * float(y.norm()), f
