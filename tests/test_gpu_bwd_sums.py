"""Rounding of the compositing backward's sums over pixels: Gaussians of pixel size
(sigma 0.55 to 0.6 px, what the dilation of 0.3 makes of every distant one), one a
tile, with the mean near the corner that the tile's four quadrants share, where a
pixel's offset from the mean is small beside its offset from a quadrant's centre.

Against float64 sums of the same records, per field. The bound is the error of the
plain form, every pixel's products rounded to float32 and added up, evaluated here
with exponential and reciprocal off by up to a unit roundoff as the device's are:
1.5 times its norm over 1000 Gaussians (whose own spread is about 1000^-0.5, 3 %;
sums in another order and fused multiply-adds change it by less than half)."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu

TX, TY = 40, 25
W, H = 16 * TX, 16 * TY
LN2 = float(np.log(2.0))


def pixel_sums(T, mean, qa, qb, qc, op, col, g, ulp):
    """The 12 gradient fields of one Gaussian per row on its tile's 256 pixels (px, py), background 0, only the
    first colour channel's upstream gradient g set; in the type T, exp2 and 1 / x off by a factor 1 + ulp[i]."""
    c = lambda x: np.asarray(x).astype(T)  # noqa: E731
    k = np.arange(256)
    px, py = c(k % 16 + 0.5), c(k // 16 + 0.5)
    col, qa, qb, qc, op, g = (c(x) for x in (col[:, None], qa[:, None], qb[:, None], qc[:, None], op[:, None], g))
    dx, dy = px - c(mean[:, :1]), py - c(mean[:, 1:])
    G = np.exp2(qa * (dx * dx) + qb * (dx * dy) + qc * (dy * dy)) * c(1.0 + ulp[0])
    al = op * G
    al = np.where(al >= T(1.0 / 255.0), al, T(0.0))
    Tf = T(1.0) - al
    Ti = Tf * (T(1.0) / (T(1.0) - al) * c(1.0 + ulp[1]))
    dal = Ti * (g * col)
    dp, w = dal * al, al * Ti
    dpx, dpy = dp * dx, dp * dy
    gx, gy = (qa + qa) * dpx + qb * dpy, qb * dpx + (qc + qc) * dpy
    on = al > 0
    out = [T(-LN2) * gx.sum(1), T(-LN2) * gy.sum(1), T(-0.5) * (dpx * dx).sum(1), -(dpx * dy).sum(1),
           T(-0.5) * (dpy * dy).sum(1), np.where(on, dal * G, T(0.0)).sum(1), (w * g).sum(1)]
    out += [np.zeros(len(col), T)] * 3 + [T(LN2) * np.abs(gx).sum(1), T(LN2) * np.abs(gy).sum(1)]
    edge = (np.abs(op * G * T(255.0) - T(1.0)) < 1e-4).any(1)
    return np.stack(out, 1).astype(np.float64), edge


@pytest.mark.parametrize("absgrad", [False, True])
def test_pixel_sized_gaussians(gpu_lib, absgrad):
    n = TX * TY
    rng = np.random.default_rng(17)
    scene = S.random_scene(n, seed=3)
    tile = np.stack([np.arange(n) % TX, np.arange(n) // TX], 1)
    at = 16.0 * tile + 8.0 + rng.uniform(-1.5, 1.5, (n, 2))
    f, z = 400.0, 40.0
    scene.means[:] = np.stack([(at[:, 0] - W / 2) / f * z, (at[:, 1] - H / 2) / f * z,
                               np.full(n, z)]).astype(np.float32).reshape(scene.means.shape)
    scene.scales[:] = (rng.uniform(0.02, 0.25, scene.scales.shape) * z / f).astype(np.float32)
    scene.opacities[:] = rng.uniform(0.3, 0.95, n).astype(np.float32)
    cam = S.Camera(f, f, W / 2.0, H / 2.0, np.eye(4, dtype=np.float32), W, H)
    opts = gpu_lib.RenderOptions(aa=False, absgrad=absgrad)
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, P = gpu_lib.bin_sort(proj, [cam], n)
    assert P == n and bool((proj.tiles == 1).all())
    out = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts)
    g = np.zeros((H, W, 3), np.float32)
    g[..., 0] = rng.standard_normal((H, W))
    res = gpu_lib.render_bwd(params, [cam], opts, proj, pairs, ranges, out["T"], out["last"],
                             torch.from_numpy(g.reshape(-1, 3)).cuda(), None, None)
    got = gpu_lib.grad2d_view(res).cpu().numpy().astype(np.float64)

    rec = proj.rec.cpu().numpy()      # the mean relative to the tile, rounded as the kernel rounds it
    mean = np.stack([(rec[:, 0] - np.float32(16) * tile[:, 0].astype(np.float32)) + rec[:, 7],
                     (rec[:, 1] - np.float32(16) * tile[:, 1].astype(np.float32)) + rec[:, 11]], 1)
    assert mean.dtype == np.float32 and np.abs(mean - 8.0).max() <= 1.6
    gt = g[..., 0].reshape(TY, 16, TX, 16).transpose(0, 2, 1, 3).reshape(n, 256)
    args = (mean, rec[:, 2], rec[:, 3], rec[:, 4], rec[:, 5], rec[:, 8], gt)
    ref, edge = pixel_sums(np.float64, *args, np.zeros((2, 1, 1)))
    plain, _ = pixel_sums(np.float32, *args, rng.uniform(-1.0, 1.0, (2, n, 256)) * 2.0 ** -24)
    ok = ~edge
    assert ok.sum() >= 0.9 * n
    for k in [0, 1, 2, 3, 4, 5, 6] + ([10, 11] if absgrad else []):
        err, bound = np.linalg.norm((got - ref)[ok, k]), np.linalg.norm((plain - ref)[ok, k])
        print(f"field {k}: error {err:.3e}, plain {bound:.3e}, of {np.linalg.norm(ref[ok, k]):.3e}")
        assert err <= 1.5 * bound, (k, err, bound)
