"""The appearance kernels at the ends of their groups of 16, chunks of 32 and 64
and workgroups of 128 and 256 Gaussians, to the bars of the larger sizes."""
import pytest

import test_gpu_appearance as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 31, 32, 33, 48, 127, 129, 255, 257])
def test_group_edges(gpu_lib, n):
    A.test_mlp_matches_oracle(gpu_lib, n)
