"""Cameras to the C array: every form of the matrix gives the same values, and a
camera changed between two calls is seen by the second."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import paper_2507_23006_amd as gs
from paper_2507_23006_amd import _lib as L

M = np.random.default_rng(3).normal(size=(4, 4))


@pytest.mark.parametrize("form", [
    lambda m: m, lambda m: m.astype(np.float32), lambda m: m.T.copy().T, lambda m: m.tolist(), lambda m: list(m),
    lambda m: torch.from_numpy(m), lambda m: tuple(map(tuple, m)), lambda m: np.round(m * 4).astype(np.int32),
    lambda m: np.vstack([m, m])])
def test_matrix_forms(form):
    m = form(M)
    cam = SimpleNamespace(fx=1.5, fy=2.5, cx=3.0, cy=4.0, viewmat=m, width=17, height=9)
    got = L.make_cameras([cam])[0]
    want = [np.float32(float(x)) for row in m for x in row][:16]
    assert [np.float32(x) for x in got.viewmat] == want
    assert (got.fx, got.fy, got.cx, got.cy, got.width, got.height) == (1.5, 2.5, 3.0, 4.0, 17, 9)


def test_short_matrix_is_refused():
    cam = SimpleNamespace(fx=1.0, fy=1.0, cx=0.0, cy=0.0, viewmat=np.eye(3), width=8, height=8)
    with pytest.raises(IndexError):
        L.make_cameras([cam])


def test_nothing_is_kept_between_calls():
    cam = SimpleNamespace(fx=1.0, fy=1.0, cx=0.0, cy=0.0, viewmat=np.eye(4), width=16, height=16)
    cams = [cam]
    assert gs.views_extent(cams) == (1, 256)
    cam.width = 33
    assert gs.views_extent(cams) == (3, 528)
    cams.append(cam)
    assert gs.views_extent(cams) == (6, 1056)
