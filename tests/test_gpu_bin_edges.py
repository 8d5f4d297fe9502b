"""Binning at the sizes where its kernels' tiles, chunks and launch forms end,
against a stable sort in NumPy of the same projected slots: every list, in order,
one for one.

Tiles of 1024 and 2048 keys, chunks of 1024 pairs, spans of 2048 slots, sorts with
and without a row scan (up to 128 tiles), compaction with and without a scan of its
counts (6144 spans)."""
import numpy as np
import pytest
import torch

import synthetic as S

pytestmark = pytest.mark.gpu


def lists(proj, n_tiles):
    tiles = proj.tiles.cpu().numpy()
    rect = proj.rect.cpu().numpy().view(np.uint32)
    key = proj.depth_key.cpu().numpy().view(np.uint32)
    mask = proj.tile_mask.cpu().numpy().view(np.uint64)
    slot = np.nonzero(tiles)[0]
    slot = slot[np.argsort(key[slot], kind="stable")]
    t0, w, tw = rect[slot, 0].astype(np.int64), (rect[slot, 1] & 0xFFFF).astype(np.int64), (rect[slot, 1] >> 16).astype(np.int64)
    whole = mask[slot] == 0
    rank, bit = np.nonzero((mask[slot][:, None] >> np.arange(64, dtype=np.uint64)) & np.uint64(1))
    for r in np.nonzero(whole)[0]:
        b = np.arange(tiles[slot[r]])
        rank, bit = np.concatenate([rank, np.full(len(b), r)]), np.concatenate([bit, b])
    tile = t0[rank] + bit // w[rank] * tw[rank] + bit % w[rank]
    o = np.lexsort((rank, tile))
    start = np.searchsorted(tile[o], np.arange(n_tiles + 1))
    return slot[rank[o]], np.stack([start[:-1], start[1:]], 1)


@pytest.mark.parametrize("n,views", [(1, 1), (63, 1), (65, 3), (1023, 1), (1024, 1), (1025, 1), (2047, 1), (2049, 2), (8191, 1),
                                     (32769, 2), (65535, 1), (65536, 1), (65537, 1), (131071, 1), (131072, 1), (131073, 1),
                                     (200_003, 2), (6144 * 1024 - 1, 2), (6144 * 1024 + 1, 2)])
def test_against_stable_sort(gpu_lib, n, views):
    scene = S.random_scene(min(n, 250_000), seed=n % 997, log_scale_mu=-4.2 if n > 5000 else -2.5)
    cams = []
    for k in range(views):
        W, H = ((75, 61), (64, 33), (40, 97))[k]
        eye = (0.7 * np.sin(2.0 * k), 0.2 * k, -4.0)
        cams.append(S.Camera(1.2 * W, 1.2 * W, W / 2.0, H / 2.0, S.look_at(eye, (0, 0, 0), up=(0, -1, 0)), W, H))
    params = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in scene.param_arrays()]
    m = params[0].shape[1]
    if n > m:      # the rest behind the cameras, the scene at both ends
        big = [torch.ones((n,) + p.shape[1:] if i == 4 else p.shape[:-1] + (n,), device="cuda") for i, p in enumerate(params)]
        big[0][2] = -50.0
        for i, p in enumerate(params):
            if i == 4:
                big[i][:m // 2], big[i][n - (m - m // 2):] = p[:m // 2], p[m // 2:]
            else:
                big[i][..., :m // 2], big[i][..., n - (m - m // 2):] = p[..., :m // 2], p[..., m // 2:]
        params = big
    opts = gpu_lib.RenderOptions(aa=False)
    proj = gpu_lib.project(*params, cams, opts)
    pairs, ranges, P = gpu_lib.bin_sort(proj, cams, n)
    vals, want = lists(proj, ranges.shape[0])
    assert P == len(vals)
    got = ranges.cpu().numpy()
    full = want[:, 1] > want[:, 0]
    assert np.array_equal(got[full], want[full]) and np.all(got[~full, 0] == got[~full, 1])
    assert np.array_equal(pairs[:P].cpu().numpy().view(np.uint32), vals)
