"""The D-SSIM kernels where their pieces end: 64 floats (21 1/3 pixels) a wave,
strips of at least 8 rows, 32 pieces to a turn of workgroups, images smaller than
the window.

The kernels blur in float32: each of the 22 FMAs of a sum rounds by 6e-8 of values
of at most 1, so variances carry about 1e-6 against C2 = 9e-4 and s about 1e-3 of
itself at worst (flat patches), far less on noise: 1e-5 for the loss, 1e-4 of the
gradient's norm."""
import numpy as np
import pytest
import torch

from oracle import ssim as OS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (3, 40), (21, 7), (22, 8), (43, 9), (64, 17), (85, 33), (129, 64), (300, 3),
                                 (700, 130)])
def test_piece_edges(gpu_lib, W, H):
    rng = np.random.default_rng(W * 1000 + H)
    x, y = (rng.uniform(0.0, 1.0, (H, W, 3)).astype(np.float32) for _ in range(2))
    xt = torch.from_numpy(x).cuda().requires_grad_(True)
    loss = gpu_lib.dssim_loss(xt, torch.from_numpy(y).cuda(), 0.2)
    loss.backward()
    ref, g = OS.dssim(x, y, 0.2)
    assert abs(loss.item() - ref) <= 1e-5
    got = xt.grad.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - g.reshape(got.shape)) <= 1e-4 * np.linalg.norm(g)
