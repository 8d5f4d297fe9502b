"""The 3D filter's sampling rate where its launches and blocks end: 24 cameras
a launch, 1024 means a block.

Rates are one float32 rounding of an FP64 value on both sides (6e-8 each);
view tests within 1e-9 of their boundary are set aside."""
import numpy as np
import pytest
import torch

import synthetic as S
from oracle import densify as OD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 1023, 1025, 5000])
@pytest.mark.parametrize("n_cams", [1, 16, 23, 24, 25, 49])
def test_launch_edges(gpu_lib, n, n_cams):
    rng = np.random.default_rng(n + n_cams)
    means = rng.uniform(-3, 3, (3, n)).astype(np.float32)
    cams = []
    for k in range(n_cams):
        eye = (4 * np.cos(k), 4 * np.sin(k), rng.uniform(-1, 1))
        cam = S.Camera(120.0 + 3 * k, 110.0, 70.0, 60.0, S.look_at(eye, (0, 0, 0), up=(0, 0, 1)), 160, 120)
        cam.near, cam.far = 1.0, 6.0
        cams.append(cam)
    rate = gpu_lib.densify.filter3d_rate(torch.from_numpy(means).cuda(), cams).cpu().numpy()
    ref, ok = OD.filter_rate(means, cams), OD.filter_rate_margin(means, cams) > 1e-9
    assert np.array_equal((rate == 0)[ok], (ref == 0)[ok])
    np.testing.assert_allclose(rate[ok], ref[ok], rtol=2e-7)
