"""Launches of few tiles whose lists would leave more states in segments of 128
positions than are kept for them (32768) take segments of 512; one state fewer and they
stay short.  Every Gaussian covers the whole image, so all lists have n entries, and
each is composited at every pixel before its stop.

Against float64 sums of the records.  Walking a list whole rounds each sum and T once
an entry; in segments a sum's terms meet in two steps, so it is rounded no more often,
and T a few times more for the folds: the error's norm over the pixels (over the
Gaussians for the gradients) is at most 1.5 times that of the same lists walked whole."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu

BG = (0.1, 0.4, 0.7)
LN2 = float(np.log(2.0))


def float64_sums(rec, W, H, last, g, pixels=None):
    """Images (at all pixels or some) and per-Gaussian gradient fields of records in list order, the first
    last[pixel] composited."""
    r = rec.double()
    mx, my, z, o, col = r[:, 0] + r[:, 7], r[:, 1] + r[:, 11], r[:, 6], r[:, 5], r[:, 8:11]
    bg = torch.tensor(BG, dtype=torch.float64, device="cuda")
    pos = torch.arange(1, len(rec) + 1, device="cuda")
    img = {k: [] for k in ("rgb", "depth", "T")}
    grad = torch.zeros(len(rec), 10, dtype=torch.float64, device="cuda")
    for pix in (torch.arange(W * H, device="cuda") if pixels is None else pixels).split(8192):
        dx, dy = (pix % W).double()[:, None] + 0.5 - mx, (pix // W).double()[:, None] + 0.5 - my
        a = o * torch.exp2(r[:, 2] * dx * dx + r[:, 3] * dx * dy + r[:, 4] * dy * dy)
        assert float(a.min()) > 1.001 / 255.0
        a = a * (pos <= last[pix, None])
        T = torch.cumprod(1.0 - a, 1)
        Tb = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
        w, Tf = a * Tb, T[:, -1:]
        img["rgb"].append(w @ col + Tf * bg)
        img["depth"].append(w @ z)
        img["T"].append(Tf[:, 0])
        gr, gd, ga = (x[pix].double() for x in g)
        gc = gr @ col.T + gd[:, None] * z
        s = gc * w
        behind = torch.flip(torch.cumsum(torch.flip(s, [1]), 1), [1]) - s + (gr @ bg)[:, None] * Tf
        dp = (Tb * gc + (ga[:, None] * Tf - behind) / (1.0 - a)) * a
        fields = [-LN2 * dp * (2 * r[:, 2] * dx + r[:, 3] * dy), -LN2 * dp * (r[:, 3] * dx + 2 * r[:, 4] * dy),
                  -0.5 * dp * dx * dx, -dp * dx * dy, -0.5 * dp * dy * dy, dp / o]
        grad += torch.stack([f.sum(0) for f in fields] + list((w.T @ gr).T) + [w.T @ gd], 1)
    return {k: torch.cat(v) for k, v in img.items()}, grad


@pytest.mark.parametrize("W,H,n,length", [(1024, 1024, 1152, 128), (1024, 1024, 1153, 512), (1024, 1024, 1500, 512),
                                          (1040, 1008, 1200, 512), (640, 368, 4500, 128), (640, 368, 4800, 512)])
def test_short_and_long(gpu_lib, W, H, n, length):
    rng = np.random.default_rng(n)
    scene = S.random_scene(n, seed=n, log_scale_mu=3.0, log_scale_sigma=0.05)
    scene.means[:] = rng.uniform(-0.02, 0.02, scene.means.shape).astype(np.float32)
    scene.opacities[:] = rng.uniform(0.0042, 0.0045, n).astype(np.float32)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(600.0, 600.0, W / 2.0, H / 2.0, vm, W, H)
    opts = gpu_lib.RenderOptions(aa=False, bg=BG)
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, P = gpu_lib.bin_sort(proj, [cam], n)
    T = ranges.shape[0]
    assert P == n * T
    seg = gpu_lib.seg_workspace([cam], pairs)
    none = torch.empty(256, dtype=torch.uint8, device="cuda")
    got = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=seg)
    whole = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=False)
    # the area starts with the offsets of the tiles' segments, the last one their number
    off = (-seg.data_ptr()) % 256
    assert int(seg[off:off + 4 * (T + 1)].view(torch.int32)[T]) == (n + length - 1) // length * T
    # (T falls by 0.4 % an entry and is known to about 2000^0.5 roundoffs, 3e-6: of the pixels whose T
    # reaches the stop threshold, one in a thousand may stop an entry apart)
    same = got["last"] == whole["last"]
    assert int((~same).sum()) <= 2e-3 * W * H
    g = [torch.from_numpy(rng.standard_normal((W * H, 3)).astype(np.float32)).cuda() * same[:, None],
         torch.from_numpy((0.2 * rng.standard_normal(W * H)).astype(np.float32)).cuda() * same,
         torch.from_numpy(rng.standard_normal(W * H).astype(np.float32)).cuda() * same]
    order = pairs[int(ranges[0, 0]):int(ranges[0, 1])].long()
    img, grad = float64_sums(proj.rec[order], W, H, whole["last"], g)
    for k, ref in img.items():
        err, bound = ((x[k][same] - ref[same]).norm() for x in (got, whole))
        assert float(err) <= 1.5 * float(bound), (k, float(err), float(bound))
    bwd = lambda out, s: gpu_lib.grad2d_view(gpu_lib.render_bwd(  # noqa: E731
        params, [cam], opts, proj, pairs, ranges, out["T"], out["last"], *g, seg=s))[order].double()
    bound = (bwd(whole, none)[:, :10] - grad).norm(dim=0)
    for area in (seg, None):      # the forward's states, and the backward's own
        err = (bwd(got, area)[:, :10] - grad).norm(dim=0)
        assert (err <= 1.5 * bound).all(), (err / bound).tolist()
