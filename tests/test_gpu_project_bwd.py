"""The projection backward's lists and chunks: 70 Gaussians in view, strewn
over N of which the rest lie behind the cameras, must get the gradients and
statistics that they get alone, and the others zeros.

N spans one chunk of 64 and its neighbours, the size from which chunks hold
256 (524288) and from which the outputs are zeroed beforehand (2097152).  Both
runs composite the same lists; only the order of the float atomics differs,
at most some 200 additions per slot: 200 x 2^-24 ~ 1.2e-5 of the sum of the
terms' sizes, taken as 1e-4 of each array's norm."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu

SEEN = 70


def view(k):
    W, H = ((40, 33), (24, 19), (31, 48))[k % 3]
    eye = (0.8 * np.sin(2.1 * k), 0.3 * k, -4.0)
    return S.Camera(1.1 * W, 1.1 * W, W / 2.0, H / 2.0, S.look_at(eye, (0.0, 0.0, 0.0), up=(0.0, -1.0, 0.0)), W, H)


def gradients(gpu_lib, arrays, cams, app, absgrad, degree):
    params = [torch.from_numpy(a).cuda().requires_grad_(True) for a in arrays]
    off = torch.from_numpy(app).cuda().requires_grad_(True) if app is not None else None
    opts = gpu_lib.RenderOptions(aa=True, absgrad=absgrad, sh_degree=degree)
    stats = gpu_lib.RenderStats()
    rgb, depth, alpha = gpu_lib.rasterize(*params, cams, opts, stats, app=off)
    rng = np.random.default_rng(5)
    w = [torch.from_numpy(rng.standard_normal(tuple(x.shape)).astype(np.float32)).cuda() for x in (rgb, depth, alpha)]
    ((w[0] * rgb).sum() + 0.2 * (w[1] * depth).sum() + (w[2] * alpha).sum()).backward()
    res = {k: p.grad for k, p in zip(("means", "scales", "quats", "opacities", "sh"), params)}
    if app is not None:
        res["app"] = off.grad
    return res, stats


@pytest.mark.parametrize("views,absgrad,with_app,degree", [(1, False, False, 3), (1, True, True, 2), (3, True, False, 3),
                                                           (9, False, True, 1)])
@pytest.mark.parametrize("n", [SEEN, 127, 129, 64 * 2048 + 1, 524287, 524288, 2097152 + 3])
def test_strewn(gpu_lib, n, views, absgrad, with_app, degree):
    rng = np.random.default_rng(n + views)
    small = S.random_scene(SEEN, seed=n % 1000 + views, log_scale_mu=-1.6)
    cams = [view(k) for k in range(views)]
    where = np.sort(rng.choice(n, SEEN, replace=False))
    app = rng.uniform(0.1, 0.4, (SEEN, 4)).astype(np.float32) if with_app else None
    arrays, large = [np.ascontiguousarray(a) for a in small.param_arrays()], []
    for k, a in enumerate(arrays):
        rows = k == 4      # coefficient rows come Gaussian by Gaussian, the rest Gaussian last
        b = np.ones((n,) + a.shape[1:] if rows else a.shape[:-1] + (n,), np.float32)
        if k == 0:
            b[2] = -50.0
        if rows:
            b[where] = a
        else:
            b[..., where] = a
        large.append(b)
    big_app = None
    if with_app:
        big_app = np.zeros((n, 4), np.float32)
        big_app[where] = app
    alone, st0 = gradients(gpu_lib, arrays, cams, app, absgrad, degree)
    strewn, st1 = gradients(gpu_lib, large, cams, big_app, absgrad, degree)
    at = torch.from_numpy(where).cuda()
    assert float(alone["sh"].norm()) > 0
    for k, a in alone.items():
        axis = 0 if k in ("sh", "app") else a.dim() - 1
        b = strewn[k].index_select(axis, at)
        assert float((a - b).norm()) <= 1e-4 * float(a.norm()), k
        rest = strewn[k].clone()
        rest.index_fill_(axis, at, 0.0)
        assert not bool(rest.any()), k
    for k in ("mean2d_grad_norm", "absgrad"):
        a, b = getattr(st0, k, None), getattr(st1, k, None)
        if a is None or not torch.is_tensor(a):
            assert b is None or not torch.is_tensor(b)
            continue
        b1 = b.index_select(1, at)
        assert float((a - b1).norm()) <= 1e-4 * float(a.norm()), k
        rest = b.clone()
        rest.index_fill_(1, at, 0.0)
        assert not bool(rest.any()), k
