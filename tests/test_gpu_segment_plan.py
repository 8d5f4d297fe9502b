"""The segment plan where its workgroups end (2048 tiles): a few long lists among
many tiles, at the start, the end and across a workgroup's end, with room for every
state, for one too few, and for none: the image must be that of whole lists.

Tolerances as for segments of any length: a few roundings of values of at most 1."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(16, 16), (32, 16384), (1024, 512), (1040, 512), (2048, 512), (2064, 1024), (8192, 1024)])
@pytest.mark.parametrize("room", ["all", "one_less", "none"])
def test_plan_edges(gpu_lib, W, H, room):
    n = 900
    rng = np.random.default_rng(W + H)
    scene = S.random_scene(n, seed=5, log_scale_mu=-6.0, log_scale_sigma=0.1)
    # a few spots all over the image, each with a long list in its tile
    spots = np.stack([rng.integers(0, W, 3), rng.integers(0, H, 3)], 1) + 0.5
    spots[0], spots[1] = (1.5, 1.5), (W - 1.5, H - 1.5)
    at = spots[rng.integers(0, 3, n)]
    z = 4.0 + rng.uniform(0, 0.5, n)
    f = 50.0
    scene.means[:] = np.stack([(at[:, 0] - W / 2) / f * z, (at[:, 1] - H / 2) / f * z, z]).astype(np.float32).reshape(
        scene.means.shape)
    scene.opacities[:] = rng.uniform(0.005, 0.02, n).astype(np.float32)
    cam = S.Camera(f, f, W / 2.0, H / 2.0, np.eye(4, dtype=np.float32), W, H)
    opts = gpu_lib.RenderOptions(aa=False)
    params = [torch.from_numpy(a).cuda() for a in scene.param_arrays()]
    proj = gpu_lib.project(*params, [cam], opts)
    pairs, ranges, _ = gpu_lib.bin_sort(proj, [cam], n)
    tiles = ranges.shape[0]
    length = (ranges[:, 1] - ranges[:, 0]).long()
    seg_len = 128 if tiles <= 4096 else 512 if tiles <= 12288 else 1024 if tiles <= 28672 else 2048
    states = int((torch.clamp((length + seg_len - 1) // seg_len, min=1) - 1).sum())
    full = gpu_lib.seg_workspace([cam], pairs)
    fixed = full.numel() - 256 - (pairs.numel() // seg_len + 1) * 6 * 1024
    keep = {"all": states, "one_less": max(states - 1, 0), "none": 0}[room]
    # aligned so that the area holds exactly `keep` states
    seg = torch.empty(fixed + keep * 6 * 1024 + 256, dtype=torch.uint8, device="cuda")
    seg = seg[(-seg.data_ptr()) % 256:][:fixed + keep * 6 * 1024]
    got = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=seg)
    ref = gpu_lib.render_fwd(proj, pairs, ranges, [cam], opts, seg=False)
    exact = room != "all" and states > 0
    for k in ("rgb", "alpha", "T", "depth"):
        d = float((got[k] - ref[k]).abs().max())
        assert d == 0.0 if exact else d <= 1e-5, k
    assert torch.equal(got["last"], ref["last"])
