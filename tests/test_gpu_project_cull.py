"""The projection's culling against every pixel in plain NumPy float64: a
Gaussian between the near and far planes whose alpha reaches 1/255 at some
pixel centre within three sigmas must keep a tile, and one whose bound misses
the image by a tile must not, for cameras that are no rotations, scenes far
from the origin, planes through the scene and images of one pixel.

Pixels within 0.1 % of the thresholds are left out: float32 parameters and
cameras enter both sides alike, and FP64 rounds far below that."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu

N = 1500


def camera(W, H, shift, linear, near, far):
    vm = np.asarray(S.look_at((1.6, -1.1, -3.3), (0.05, 0.1, 0.0), up=(0.3, -1, 0.2)), np.float64).copy()
    vm[:3, :3] = linear @ vm[:3, :3]
    vm[:3, 3] = linear @ vm[:3, 3] - vm[:3, :3] @ shift
    f = 1.2 * max(W, 8)
    cam = S.Camera(f, f, W / 2.0 + 0.3, H / 2.0, vm.astype(np.float32), W, H)
    cam.near, cam.far = near, far
    return cam


@pytest.mark.parametrize("views", [1, 3])
@pytest.mark.parametrize("case", ["plain", "scaled", "sheared", "far_away", "planes", "pixel"])
def test_nothing_seen_is_dropped(gpu_lib, case, views):
    scene = S.random_scene(N, seed=11, log_scale_mu=-3.0, log_scale_sigma=1.2)
    shift, linear, near, far, W, H = np.zeros(3), np.eye(3), 0.01, 1e10, 53, 37
    if case == "scaled":
        linear = np.eye(3) * 2.5
    if case == "sheared":
        linear = np.array([[1.0, 0.4, 0.0], [0.0, 0.8, 0.3], [0.1, 0.0, 1.3]])
    if case == "far_away":
        shift = np.array([3000.0, -2000.0, 500.0])
    if case == "planes":
        near, far = 3.2, 3.9
    if case == "pixel":
        W, H = 1, 1
    arrays = [np.ascontiguousarray(a) for a in scene.param_arrays()]
    arrays[0] = (arrays[0].astype(np.float64) + shift[:, None]).astype(np.float32)
    cams = [camera(W, H, shift, linear, near, far) for _ in range(views)]
    opts = gpu_lib.RenderOptions(aa=False)
    proj = gpu_lib.project(*[torch.from_numpy(a).cuda() for a in arrays], cams, opts)
    tiles = proj.tiles.cpu().numpy().reshape(views, N)
    mu, sc, q, op = (a.astype(np.float64) for a in arrays[:4])
    op = op.reshape(-1)
    w, x, y, z = q / np.linalg.norm(q, axis=0)
    R = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                  [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                  [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]).transpose(2, 0, 1)
    M = R * sc.T[:, None, :]
    must_total = 0
    for v, cam in enumerate(cams):
        vm = cam.viewmat.astype(np.float64)
        t = vm[:3, :3] @ mu + vm[:3, 3:]
        u, vv = t[0] / t[2], t[1] / t[2]
        fx, fy = np.float64(np.float32(cam.fx)), np.float64(np.float32(cam.fy))
        cx, cy = np.float64(np.float32(cam.cx)), np.float64(np.float32(cam.cy))
        uc = np.clip(u, -(cx + 0.15 * W) / fx, (W - cx + 0.15 * W) / fx)
        vc = np.clip(vv, -(cy + 0.15 * H) / fy, (H - cy + 0.15 * H) / fy)
        J = np.zeros((N, 2, 3))
        J[:, 0, 0], J[:, 0, 2], J[:, 1, 1], J[:, 1, 2] = fx / t[2], -fx * uc / t[2], fy / t[2], -fy * vc / t[2]
        T = J @ vm[:3, :3] @ M
        cov = T @ T.transpose(0, 2, 1) + np.eye(2) * np.float64(np.float32(opts.dilation))
        conic = np.linalg.inv(cov)
        px, py = np.meshgrid(np.arange(W) + 0.5, np.arange(H) + 0.5)
        dx, dy = px.reshape(-1)[None] - (fx * u + cx)[:, None], py.reshape(-1)[None] - (fy * vv + cy)[:, None]
        q2 = conic[:, 0, 0, None] * dx * dx + 2 * conic[:, 0, 1, None] * dx * dy + conic[:, 1, 1, None] * dy * dy
        inside = (t[2] > near * 1.001) & (t[2] < far * 0.999)
        hit = ((op[:, None] * np.exp(-0.5 * q2) >= 1.001 / 255) & (q2 <= 8.99)).any(1)
        must = inside & hit
        must_total += int(must.sum())
        assert np.all(tiles[v][must] > 0), (case, np.nonzero(must & (tiles[v] == 0))[0][:5])
        radius = 3 * np.sqrt(np.linalg.eigvalsh(cov)[:, 1]) + 18
        mx, my = fx * u + cx, fy * vv + cy
        out = (t[2] < near * 0.999) | (t[2] > far * 1.001) | (op < 0.999 / 255)
        out |= (mx + radius < 0) | (mx - radius > W + 16) | (my + radius < 0) | (my - radius > H + 16)
        assert np.all(tiles[v][out] == 0), (case, np.nonzero(out & (tiles[v] > 0))[0][:5])
    assert must_total > (0 if case == "pixel" else 20)
