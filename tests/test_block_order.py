"""The 32 output blocks that are resident together on one XCD (host arithmetic): a patch of 12 operand tiles, or
at the end of a column of patches two pieces of one, whatever the number of rows."""
import os

import pytest

from paper_2506_13996_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2506_13996_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


@pytest.mark.parametrize("tiles_r,tiles_c", [(64, 16), (63, 16), (62, 24), (61, 16), (23, 56), (47, 104), (16, 496),
                                             (63, 496), (33, 32)])
def test_runs_are_patches(tiles_r, tiles_c):
    n = B.alst_debug_block_tile(tiles_r, tiles_c, 1, 0)[0]
    runs = {}
    for bid in range(n):
        _, part, tr, tc = B.alst_debug_block_tile(tiles_r, tiles_c, 1, bid)
        if part >= 0:
            runs.setdefault((bid // 256, bid % 8), []).append((tr, tc))
    full = [r for r in runs.values() if len(r) == 32]
    assert len(full) >= (tiles_r * tiles_c // 256) * 8
    wide = [r for r in full if len({tr for tr, _ in r}) + len({tc for _, tc in r}) > 12]
    # (columns of patches are 8 blocks wide here, and one run may straddle the end of each)
    assert len(wide) <= tiles_c // 8 - 1, (len(wide), len(full))
    for r in full:
        if r not in wide:                    # the sharers of a tile are all there: rows x columns
            assert len({tr for tr, _ in r}) * len({tc for _, tc in r}) == 32


@pytest.mark.parametrize("tiles_r,tiles_c,whole_rows", [(63, 16, True), (31, 8, True), (23, 8, True),
                                                        (62, 24, False), (61, 16, False), (17, 8, False)])
def test_a_last_round(tiles_r, tiles_c, whole_rows):
    """Half a round and more: an XCD gets whole rows of a patch (8 blocks), so that their sharers stay
    together, where that leaves none with more than a tenth above the mean; else the blocks are spread one
    by one."""
    left = tiles_r * tiles_c % 256
    assert left >= 128
    n = B.alst_debug_block_tile(tiles_r, tiles_c, 1, 0)[0]
    per_xcd = [[] for _ in range(8)]
    for bid in range(n - 256, n):
        _, part, tr, tc = B.alst_debug_block_tile(tiles_r, tiles_c, 1, bid)
        if part >= 0:
            per_xcd[bid % 8].append((tr, tc // 8))
    lengths = [len(b) for b in per_xcd]
    assert sum(lengths) == left and max(lengths) * 8 <= 1.1 * left
    assert whole_rows == all(blocks.count(row) == 8 for blocks in per_xcd for row in set(blocks))
    assert max(lengths) - min(lengths) <= (8 if whole_rows else 1)
