"""Bytes of the segment area: a state is 6 KB; launches of few tiles take a state for
each 128 pairs, but no more than 32768 of them (or one for each 512 pairs, what larger
launches took all along)."""
import pytest

from paper_2507_23006_amd import _lib as L


@pytest.mark.parametrize("tiles", [1, 80, 920, 4096])
@pytest.mark.parametrize("pairs", [0, 127, 128, 100_000, 4_194_175, 4_194_303, 4_200_000, 16_777_216, 24_000_000,
                                   1_000_000_000])
def test_few_tiles(tiles, pairs):
    lib = L.load()
    state = 6 * 256 * 4
    states = (lib.gs_seg_workspace_size(tiles, pairs) - lib.gs_seg_workspace_size(tiles, 0)) // state + 1
    assert states >= min(pairs // 128 + 1, 32768)
    assert states <= max(min(pairs // 128 + 1, 32768), pairs // 512 + 1)


@pytest.mark.parametrize("tiles,length", [(4097, 512), (12288, 512), (12289, 1024), (28672, 1024), (28673, 2048)])
def test_more_tiles(tiles, length):
    lib = L.load()
    for pairs in (100_000, 24_000_000):
        assert lib.gs_seg_workspace_size(tiles, pairs) - lib.gs_seg_workspace_size(tiles, 0) == pairs // length * 6144
