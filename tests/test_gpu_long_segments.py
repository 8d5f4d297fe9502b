"""Lists of 2200 entries that no pixel stops in, in launches whose segments have 512,
1024 and 2048 positions: the same records and lists, the same quadrant of pixels.

A longer segment must not round more: the forward adds up parts of 512 positions in
each, and the backward divides T by reciprocals good to half an ulp where its walks are
longer than 512 (2048^0.5 of them add up to no more than 512 that may all be off by an
ulp the same way).  Against float64 sums of the records: at most 1.5 times the error of
the launch in segments of 512.  The pixels' alphas are alike and so are their errors: a
field of a seed is about one sample, and the root mean square over six seeds and the
four (six) fields made of w (dp) spreads by a seventh (an eighth) on either side."""
import numpy as np
import pytest
import torch

import synthetic as S
from test_gpu_segment_states import BG, float64_sums

pytestmark = pytest.mark.gpu


def errors(gs, W, H, seed):
    n = 2200
    rng = np.random.default_rng(seed)
    scene = S.random_scene(n, seed=seed, log_scale_mu=-0.5, log_scale_sigma=0.02)
    scene.means[:] = rng.uniform(-0.005, 0.005, scene.means.shape).astype(np.float32)
    scene.opacities[:] = rng.uniform(0.00405, 0.0042, n).astype(np.float32)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(600.0, 600.0, 804.0, 516.0, vm, W, H)      # in the middle of a quadrant
    opts = gs.RenderOptions(aa=False, bg=BG)
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gs.project(*params, [cam], opts)
    pairs, ranges, _ = gs.bin_sort(proj, [cam], n)
    tile = 516 // 16 * ((W + 15) // 16) + 804 // 16
    order = pairs[int(ranges[tile, 0]):int(ranges[tile, 1])].long()
    assert len(order) == n
    seg = gs.seg_workspace([cam], pairs)
    out = gs.render_fwd(proj, pairs, ranges, [cam], opts, seg=seg)
    y, x = torch.meshgrid(torch.arange(512, 520, device="cuda"), torch.arange(800, 808, device="cuda"), indexing="ij")
    pixels = (y * W + x).ravel()
    assert bool((out["last"][pixels] == n).all())
    g = [torch.zeros((W * H, 3), device="cuda"), torch.zeros(W * H, device="cuda"), torch.zeros(W * H, device="cuda")]
    for t in g:
        t[pixels] = torch.from_numpy(rng.standard_normal(t[pixels].shape).astype(np.float32)).cuda()
    img, grad = float64_sums(proj.rec[order], W, H, out["last"], g, pixels)
    got = gs.grad2d_view(gs.render_bwd(params, [cam], opts, proj, pairs, ranges, out["T"], out["last"], *g, seg=seg))
    err = (got[order][:, :10].double() - grad).norm(dim=0) / grad.norm(dim=0)
    images = torch.stack([(out[k][pixels] - img[k]).norm() / img[k].norm() for k in ("rgb", "depth")])
    return torch.cat([images, err]).cpu().numpy()


@pytest.mark.parametrize("W,H", [(2112, 2000), (3008, 3000)])
def test_no_further_from_float64(gpu_lib, W, H):
    a, b = (np.mean([errors(gpu_lib, *s, seed) ** 2 for seed in range(6)], 0) for s in ((1600, 1072), (W, H)))
    for name, part in (("images", slice(0, 2)), ("dp", slice(2, 8)), ("w", slice(8, 12))):
        ratio = np.sqrt(b[part].mean() / a[part].mean())
        print(name, "segments of 512: %.2e" % np.sqrt(a[part].mean()), "longer / 512: %.2f" % ratio)
        assert ratio <= 1.5, name
