"""Which launches are cut into tiles of several heights (no GPU): the library's own rules, asked through the built library."""
import ctypes

import pytest

from gpu_util import gemm_path
from paper_2605_21603_amd import binding as B


def fold_tiles(rows, n, k, n_cus=0):
    """m tiles of 96, 128 and 160 rows of a launch with folded planes, None where it keeps one height."""
    tiles, f = (ctypes.c_int * 3)(), B.lib()._ZN3dyn13gemm_fold_cutERKNS_8GemmPathEiiiiPNS_7FoldCutE
    f.argtypes, f.restype = [ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.c_void_p], ctypes.c_bool
    p = gemm_path(rows, n, k)
    return list(tiles) if p.folded and f(ctypes.byref(p), rows, n, k, n_cus, tiles) else None


@pytest.mark.parametrize("n,k", [(8192, 28672), (10240, 16384)])
def test_large_weights_are_not_read_again_for_a_part_of_a_round(n, k):
    """Weights of more than 256 MiB: the last of several heights would read them from memory once more, for less work than that takes if
    its tiles are less than a round (512).  All tiles at once walk them together."""
    cuts = 0
    for rows in range(513, 6000, 41):
        tiles = fold_tiles(rows, n, k)
        assert fold_tiles(rows, n, k, n_cus=128) is None
        if tiles:
            m_tiles = n // 128 * sum(tiles)
            last = n // 128 * next(t for t in tiles if t)             # the lowest tiles run last
            assert m_tiles <= 512 or last == m_tiles or last >= 512, (rows, tiles)
            cuts += 1
    assert cuts > 30


def test_weights_of_the_last_level_cache_are_cut_by_their_rounds_alone():
    tiles, f = (ctypes.c_int * 3)(), B.lib()._ZN3dyn8fold_cutERKNS_8GemmPathEiiPNS_7FoldCutE
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p], ctypes.c_bool
    for n, k in ((8192, 7168), (6144, 4096), (4096, 14336)):
        for rows in range(513, 4200, 53):
            p = gemm_path(rows, n, k)
            assert fold_tiles(rows, n, k) == (list(tiles) if p.folded and f(ctypes.byref(p), rows, n, tiles) else None)


def test_the_heights_of_a_cut_hold_its_rows():
    cuts = 0
    for n in (1024, 3072, 4096, 8192, 13824):
        for k in (1024, 4096, 14336, 28672):
            for rows in range(513, 6000, 97):
                tiles = fold_tiles(rows, n, k)
                if tiles:
                    cuts += 1
                    assert 0 <= 32 * sum((3 + i) * t for i, t in enumerate(tiles)) - rows < 96
    assert cuts > 200


@pytest.mark.parametrize("hidden,inter", [(2048, 8192), (2560, 6912), (1024, 4096)])
def test_gate_up_folds_its_planes_on_few_cus_on_the_tallest_tiles_alone(hidden, inter):
    """One round of tiles on the whole chip is several on a partition: below 128 CUs planes stay spread over the workgroups, but for 256-row tiles."""
    tile, taken = B.lib()._ZN3dyn14gate_fold_rowsEiii, B.lib()._ZN3dyn15gate_fold_takenEiiii
    heights = set()
    for rows in range(64, 600, 7):
        mt = tile(rows, 2 * inter, hidden)
        heights.add(mt)
        assert (mt > 0) == (128 < rows <= 512)
        assert [taken(rows, 2 * inter, hidden, n) & 0xff for n in (0, 256, 128, 120, 64)] == [mt > 0] * 3 + [mt == 256] * 2
    assert len(heights) >= 3


@pytest.mark.parametrize("hidden,inter,low", [(4096, 4096, True), (5120, 8192, True), (8192, 4096, False), (8192, 8192, False)])
def test_gate_up_of_deep_weights_folds_its_planes_on_tall_tiles_alone(hidden, inter, low):
    """A low tile moves 128 W rows a stage for its 64 or 128 rows, and deeper than 5120 that is more than the planes' way through memory."""
    tile = B.lib()._ZN3dyn14gate_fold_rowsEiii
    heights = {tile(rows, 2 * inter, hidden) for rows in range(129, 513)} - {0}
    assert (min(heights, default=256) < 192) == low
    assert tile(513, 2 * inter, hidden) == tile(128, 2 * inter, hidden) == 0
