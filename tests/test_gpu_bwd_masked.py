"""A pixel's upstream gradient of alpha reaches only the entries composited there: an
infinity or a NaN at pixels without any (d log(alpha) or d(depth / alpha) where alpha
is 0) leaves every gradient as it is with 0 there, though the pixel's quadrant holds
other entries.

Two runs of the same sums differ by the order of their float atomics, a few dozen
roundings of 6e-8 per slot: 1e-5 of each field's norm."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("absgrad", [False, True])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_alpha_gradient_where_nothing_is_composited(gpu_lib, value, absgrad):
    W, H, n = 130, 93, 400
    rng = np.random.default_rng(4)
    scene = S.random_scene(n, seed=12, log_scale_mu=-3.2, log_scale_sigma=0.4)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(110.0, 110.0, W / 2.0, H / 2.0, vm, W, H)
    opts = gpu_lib.RenderOptions(aa=False, absgrad=absgrad, bg=(0.2, 0.5, 0.1))
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, _ = gpu_lib.bin_sort(proj, [cam], n)
    out = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts)
    empty = out["last"] == 0
    quads = empty[:W * (H // 8 * 8)].view(H // 8, 8, W)[:, :, :W // 8 * 8].reshape(H // 8, 8, W // 8, 8).float().mean((1, 3))
    assert int(((quads > 0) & (quads < 1)).sum()) > 30      # quadrants with both kinds of pixels
    g = [torch.from_numpy(rng.standard_normal((W * H, 3)).astype(np.float32)).cuda(),
         torch.from_numpy(rng.standard_normal(W * H).astype(np.float32)).cuda(),
         torch.from_numpy(rng.standard_normal(W * H).astype(np.float32)).cuda()]
    grads = []
    for at_empty in (0.0, value):
        g[2][empty] = at_empty
        res = gpu_lib.render_bwd(params, [cam], opts, proj, pairs, ranges, out["T"], out["last"], *g)
        grads.append({**{k: res[k] for k in ("means", "scales", "quats", "opacities", "sh")},
                      "grad2d": gpu_lib.grad2d_view(res)[proj.tiles > 0][:, :12 if absgrad else 10].clone()})
    for k, ref in grads[0].items():
        assert torch.isfinite(ref).all() and float(ref.norm()) > 0.0
        assert torch.isfinite(grads[1][k]).all(), k
        if k == "grad2d":
            for f in range(ref.shape[1]):
                assert float((grads[1][k][:, f] - ref[:, f]).norm()) <= 1e-5 * float(ref[:, f].norm()), f
