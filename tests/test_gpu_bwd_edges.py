"""The compositing backward at the sizes where its batches and chunks end:
per-slot 2D gradients (AbsGS sums included) of lists of 1 to 600 entries on a
ragged image, against the same sums in plain NumPy float64 from the records.

The float32 walk recovers T over up to 600 divisions (about 3 unit roundoffs
each, 1e-4 in all at the deepest entry, far less where the weight is) and its
differences g.c - S cancel a digit at most: 2e-4 of each field's norm."""
import numpy as np
import pytest
import torch

import synthetic as S
from gpu_util import decode_records

pytestmark = pytest.mark.gpu

W, H = 24, 19


def reference(mean, conic, op, rgb, z, bg, g_rgb, g_d, g_a):
    px, py = np.meshgrid(np.arange(W) + 0.5, np.arange(H) + 0.5)
    dx, dy = px.reshape(-1, 1) - mean[:, 0], py.reshape(-1, 1) - mean[:, 1]
    G = np.exp(-0.5 * (conic[:, 0] * dx * dx + conic[:, 2] * dy * dy) - conic[:, 1] * dx * dy)
    raw = op * G
    a = np.minimum(raw, 0.99)
    a = np.where(a >= 1.0 / 255.0, a, 0.0)
    T = np.cumprod(1.0 - a, axis=1)
    a = np.where(T >= 1e-4, a, 0.0)
    T = np.cumprod(1.0 - a, axis=1)
    Tb = np.concatenate([np.ones((len(T), 1)), T[:, :-1]], axis=1)
    w, Tf = a * Tb, T[:, -1:]
    gc = g_rgb @ rgb.T + g_d[:, None] * z
    behind = np.cumsum((gc * w)[:, ::-1], axis=1)[:, ::-1] - gc * w + (g_rgb @ bg)[:, None] * Tf
    da = Tb * gc + (g_a[:, None] * Tf - behind) / (1.0 - a)
    dp = np.where((a > 0.0) & (raw < 0.99), da * a, 0.0)
    mx, my = dp * (conic[:, 0] * dx + conic[:, 1] * dy), dp * (conic[:, 1] * dx + conic[:, 2] * dy)
    out = [mx, my, -0.5 * dp * dx * dx, -dp * dx * dy, -0.5 * dp * dy * dy, dp / op]
    out += [w * g_rgb[:, c:c + 1] for c in range(3)] + [w * g_d[:, None], np.abs(mx), np.abs(my)]
    return np.stack([f.sum(0) for f in out], 1)


@pytest.mark.parametrize("absgrad", [False, True])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 130, 600])
def test_list_lengths(gpu_lib, n, absgrad):
    rng = np.random.default_rng(n)
    scene = S.random_scene(n, seed=n, log_scale_mu=-1.2, log_scale_sigma=0.6)
    scene.opacities[:] = rng.uniform(0.02, 0.3 if n > 100 else 0.9, n).astype(np.float32)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(30.0, 30.0, W / 2.0, H / 2.0, vm, W, H)
    opts = gpu_lib.RenderOptions(aa=False, absgrad=absgrad, bg=(0.1, 0.4, 0.7))
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, _ = gpu_lib.bin_sort(proj, [cam], n)
    out = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts)
    g = [rng.standard_normal((W * H, 3)), rng.standard_normal(W * H) * 0.2, rng.standard_normal(W * H)]
    g = [x.astype(np.float32) for x in g]
    res = gpu_lib.render_bwd(params, [cam], opts, proj, pairs, ranges, out["T"], out["last"],
                             *[torch.from_numpy(x).cuda() for x in g])
    seen = (proj.tiles > 0).cpu().numpy()
    order = np.argsort(proj.depth_key.cpu().numpy().view(np.uint32), kind="stable")
    order = order[seen[order]]
    mean, conic, op, rgb, z = (x[order] for x in decode_records(proj.rec.cpu().numpy()))
    ref = reference(mean, conic, op, rgb, z, np.array(opts.bg), *[x.astype(np.float64) for x in g])
    got = gpu_lib.grad2d_view(res).cpu().numpy()[order].astype(np.float64)
    for f in range(12 if absgrad else 10):
        err = np.linalg.norm(got[:, f] - ref[:, f]) / max(np.linalg.norm(ref[:, f]), 1e-30)
        assert err <= 2e-4, (f, err)
