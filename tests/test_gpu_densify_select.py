"""The budgeted selection where its blocks, histograms and ties end, against a
stable sort in NumPy: 1024 Gaussians a block, 11 + 11 + 10 bits of the key, and
equal scores that the budget cuts (the first in index order grow).

Scores are chosen exactly (tau = 1 everywhere, float32 means), so the decisions
have no rounding and must match one for one."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 4096, 5000, 70_001])
@pytest.mark.parametrize("scores", ["distinct", "few", "one", "low_bits", "sparse"])
def test_against_stable_sort(gpu_lib, n, scores):
    D = gpu_lib.densify
    rng = np.random.default_rng(n)
    mean = np.full(n, 0.5, np.float32)
    on = rng.random(n) < (0.02 if scores == "sparse" else 0.7)
    k = int(on.sum())
    if scores in ("distinct", "sparse"):
        mean[on] = rng.uniform(1.5, 1e6, k).astype(np.float32)
    elif scores == "few":
        mean[on] = rng.choice(np.float32([1.5, 2.0, 7.0, 7.5, 1e20]), k)
    elif scores == "one":
        mean[on] = 3.0
    else:
        mean[on] = (np.float32(2.0).view(np.uint32) + rng.integers(0, 40, k).astype(np.uint32)).view(np.float32)
    opac = rng.uniform(0.0, 1.0, n).astype(np.float32)
    scales = np.exp(rng.normal(-2.3, 0.5, (3, n))).astype(np.float32)
    st = D.DensifyStats(n, "cuda")
    st.accum.copy_(torch.from_numpy(mean))
    st.count.fill_(1)
    args = [torch.from_numpy(a).cuda() for a in (np.zeros((3, n), np.float32), scales, opac)]
    pruned = opac < np.float32(0.1)
    cand = np.nonzero(on & ~pruned)[0]
    order = cand[np.argsort(-mean[cand], kind="stable")]
    kind = np.where(scales.max(0) > np.float32(0.1), D.SPLIT, D.CLONE)
    E, left = len(cand), n - int(pruned.sum())
    for room in sorted({0, 1, E // 3, E // 2, max(E - 1, 0), E, E + 5}):
        p = D.DensifyParams((0, 0, 0), (0, 0, 0), tau_min=1.0, eta=1.0, d_max=1.0, prune_opacity=0.1, split_scale=0.1,
                            budget=left + room)
        act, counts = D.select(st, *args, p)
        want = np.where(pruned, D.PRUNE, D.KEEP)
        want[order[:room]] = kind[order[:room]]
        assert np.array_equal(act.cpu().numpy(), want), (room, E)
        assert counts == {"candidates": E, "pruned": int(pruned.sum()), "grown": min(room, E), "room": room}
