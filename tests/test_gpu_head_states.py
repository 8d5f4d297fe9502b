"""Segment states that the compositing forward's head writes (lists up to 1024
positions in segments of 128): the colour of a deep segment is a small part of the sum
so far, and has to keep its own precision for the backward that starts from it.

Gradients of such lists against float64 sums of the records, T falling to 0.004, on an
image of one quadrant, so that no two sums meet in an atomic. A walk from a state
divides T by fewer entries than a walk of the whole list and carries fewer sums, so its
error is at most the whole walk's; norms of errors that 64 pixels share spread by about
a tenth on either side: 1.5 times."""
import numpy as np
import pytest
import torch

import synthetic as S
from test_gpu_segment_states import BG, float64_sums

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [260, 640, 1000, 1024])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_gradients_from_head_states(gpu_lib, n, seed):
    W = H = 8
    rng = np.random.default_rng(1000 * seed + n)
    scene = S.random_scene(n, seed=seed, log_scale_mu=-2.0, log_scale_sigma=0.05)
    scene.means[:] = rng.uniform(-0.02, 0.02, scene.means.shape).astype(np.float32)
    lo = 0.0048
    scene.opacities[:] = rng.uniform(lo, 2.0 * 5.5 / n - lo, n).astype(np.float32)
    vm = np.eye(4, dtype=np.float32)
    vm[2, 3] = 4.0
    cam = S.Camera(600.0, 600.0, W / 2.0, H / 2.0, vm, W, H)
    opts = gpu_lib.RenderOptions(aa=False, bg=BG)
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, P = gpu_lib.bin_sort(proj, [cam], n)
    assert P == n and ranges.shape[0] == 1
    seg = gpu_lib.seg_workspace([cam], pairs)
    none = torch.empty(256, dtype=torch.uint8, device="cuda")
    got = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=seg)
    whole = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=False)
    assert torch.equal(got["last"], whole["last"]) and int(whole["last"].min()) == n
    g = [torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda() for s in ((W * H, 3), W * H, W * H)]
    order = pairs.long()
    _, grad = float64_sums(proj.rec[order], W, H, whole["last"], g)
    bwd = lambda out, s: gpu_lib.grad2d_view(gpu_lib.render_bwd(  # noqa: E731
        params, [cam], opts, proj, pairs, ranges, out["T"], out["last"], *g, seg=s))[order].double()
    bound = (bwd(whole, none)[:, :10] - grad).norm(dim=0)
    err = (bwd(got, seg)[:, :10] - grad).norm(dim=0)
    print("error / whole walk's:", ["%.2f" % x for x in (err / bound).tolist()])
    assert (err <= 1.5 * bound).all()
