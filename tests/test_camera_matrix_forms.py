"""Forms of a camera's matrix that are read element by element: each gives the values
of its elements, and what is no matrix of numbers is refused."""
import warnings
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2507_23006_amd import _lib as L

M = np.random.default_rng(8).normal(size=(4, 4))


def convert(m):
    cam = SimpleNamespace(fx=1.5, fy=2.5, cx=3.0, cy=4.0, viewmat=m, width=17, height=9)
    with warnings.catch_warnings():      # (numpy: an imaginary part dropped, a one-element array as a number)
        warnings.simplefilter("ignore")
        return np.array(list(L.make_cameras([cam])[0].viewmat))


@pytest.mark.parametrize("form", [
    lambda: M[:, :, None], lambda: torch.from_numpy(M)[:, :, None], lambda: M.astype(complex),
    lambda: torch.from_numpy(M).to(torch.complex128), lambda: torch.from_numpy(M).to_sparse(),
    lambda: [[np.array(x) for x in row] for row in M], lambda: M.astype(str), lambda: M.astype(object),
    lambda: torch.from_numpy(M).requires_grad_(), lambda: torch.nn.Parameter(torch.from_numpy(M)),
    lambda: np.ma.masked_array(M, np.zeros((4, 4), bool))])
def test_elementwise_forms(form):
    assert np.array_equal(convert(form()), M.astype(np.float32).ravel())


def test_masked_element():
    want = M.astype(np.float32)
    want[M > 1.0] = np.nan
    assert (M > 1.0).any()
    assert np.array_equal(convert(np.ma.masked_array(M, M > 1.0)), want.ravel(), equal_nan=True)


@pytest.mark.parametrize("form", [lambda: np.matrix(M), lambda: memoryview(M), lambda: M[None], lambda: M.ravel()])
def test_refused_forms(form):
    with pytest.raises((TypeError, NotImplementedError)):
        convert(form())
