"""The chunks of cross-entropy launches (host arithmetic): for every number of dense rows a chunk may turn out
to have, its launches hold the blocks that the device chooses, and partial products are added up whenever
there are any."""
import os
import random

import pytest

from paper_2506_13996_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2506_13996_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def _check(N, H, V, tile, flags, chunk, dense):
    i = B.alst_debug_ce_chunk(N, H, V, tile, flags, chunk, dense)
    case = (N, H, V, tile, flags, chunk, dense, i.ranges, i.added_up, i.dhidden_blocks, i.dhidden_grid)
    assert i.ranges == 1 or i.added_up, case
    assert i.dhidden_blocks <= i.dhidden_grid, case
    assert i.largest_grid < 1 << 24, case              # workgroups of 256, fewer than 2^32 threads
    assert i.largest_grid >= max(i.gather_grid, i.dhidden_grid, i.dw_grid), case
    # the gathering launch: the rows, those who look for ignored tokens and, unless that is too many, those who transpose W
    rows, zeroes = -(-i.rows // 256) * 256, min(-(-N // 16), 32768) if chunk == 0 else 0
    pieces = -(-V // 64) * -(-H // 64) if chunk == 0 else 0
    assert i.transposed_apart == (rows + zeroes + pieces > (1 << 24) - 256), case
    assert i.gather_grid == rows + zeroes + (0 if i.transposed_apart else pieces), case
    # small blocks are at most one round of the compute units, with dW's if these are in the same launch
    if i.dhidden_columns:
        assert i.dhidden_grid == 256 and i.dhidden_blocks + (i.dw_blocks if i.together else 0) <= 256, case
    if i.dw_columns:
        assert i.dw_blocks <= 256, case
    assert i.dw_blocks <= i.dw_grid or i.together or i.dw_blocks == 0, case
    if i.together:
        assert i.dhidden_columns == i.dw_columns != 0 and i.dw_grid == 0, case
    return i


# more than 4096 row blocks, of which the valid rows are few or many
@pytest.mark.parametrize("N,H,V", [(1_048_832, 8, 1024), (1_048_832, 8, 2048), (1_200_000, 64, 4096),
                                   (1_100_000, 64, 32000), (1_100_000, 1600, 50257), (16_776_960, 8, 40)])
def test_long_chunks(N, H, V):
    for dense in [0, 1, 500, 3000, 8000, 12_000, 50_000, 213_000, *range(1000, N, N // 400), N]:
        i = B.alst_debug_ce_chunk(N, H, V, N, 0, 0, 0)
        _check(N, H, V, N, 0, 0, min(dense, i.rows))
    assert any(B.alst_debug_ce_chunk(N, H, V, N, 0, 0, d).ranges > 1 for d in (500, 3000, 8000)) or V < 1024


def test_random_shapes():
    rng = random.Random(11)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    for _ in range(1500):
        N, H, V = log(1, 1 << 24), log(8, 6000) // 8 * 8, log(1, 300_000)
        tile, flags = log(1, 1 << 24), rng.choice([0, B.ALST_FLAG_TILE_SCRATCH])
        first = B.alst_debug_ce_chunk(N, H, V, tile, flags, 0, 0)
        for _ in range(4):
            _check(N, H, V, tile, flags, 0, rng.randint(0, first.rows))
        if first.rows < N:
            second = B.alst_debug_ce_chunk(N, H, V, tile, flags, 1, 0)
            assert second.first == first.rows
            _check(N, H, V, tile, flags, 1, rng.randint(0, second.rows))


@pytest.mark.parametrize("N,H,V,tile,rows", [
    (131072, 4096, 128256, 4096, 4096), (131072, 1024, 200064, 4096, 16384), (131072, 4096, 65536, 4096, 16384),
    (20000, 8192, 128256, 2048, 4096), (20000, 2048, 128256, 8192, 8192), (12000, 4096, 98304, 300, 4096),
    (5000, 4096, 128256, 2048, 5000), (9300, 4096, 128256, 2048, 4096),
])
def test_chunks_of_a_long_vocabulary(N, H, V, tile, rows):
    """About one round of dHidden's 256 x 256 blocks; a last chunk up to a quarter longer."""
    at, k, lengths = 0, 0, []
    while at < N:
        i = _check(N, H, V, tile, 0, k, 0)
        assert i.first == at and i.group0 <= at
        _check(N, H, V, tile, 0, k, i.rows)
        lengths.append((i.group0, i.rows))
        at, k = at + i.rows, k + 1
    assert at == N and lengths[0][1] == rows
    for (group, n), (after, _) in zip(lengths, lengths[1:] + [(-1, 0)]):
        assert n == rows if group == after else n <= rows + rows // 4      # (a group's last chunk)


@pytest.mark.parametrize("N,H,V,apart", [(4096, 4096, 128256, 0), (8192, 8192, 8380000, 0), (4096, 8192, 8388608, 1)])
def test_the_transposition_is_a_launch_of_its_own_where_a_grid_ends(N, H, V, apart):
    assert _check(N, H, V, 2048, 0, 0, 0).transposed_apart == apart
    if N > 4096:
        assert _check(N, H, V, 2048, 0, 1, 0).transposed_apart == 0


def test_small_blocks_for_every_number_of_rows():
    """Every number of dense rows of short calls around the ends of the rules, where the ranges change with the rows."""
    seen = set()
    for N, H, V in [(512, 256, 4096), (512, 512, 4096), (1024, 256, 2048), (1024, 72, 500), (300, 520, 1000), (2048, 256, 1000),
                    (256, 64, 20000), (700, 2304, 2304), (1000, 64, 3000), (200, 512, 4000), (1024, 512, 2048), (100, 2304, 2304),
                    (3000, 256, 1500)]:
        for tile in (128, N):
            at, k = 0, 0
            while at < N:
                rows = B.alst_debug_ce_chunk(N, H, V, tile, 0, k, 0).rows
                for dense in range(0, rows + 1, 1 if rows < 400 else 7):
                    i = _check(N, H, V, tile, 0, k, dense)
                    seen.add((i.dhidden_columns, i.dw_columns, i.together))
                at, k = at + rows, k + 1
    assert seen >= {(64, 64, 1), (128, 128, 1), (64, 128, 0), (128, 64, 0), (128, 0, 0), (0, 64, 0), (0, 0, 0)}, seen


@pytest.mark.parametrize("N,H,V,together", [
    (512, 256, 4096, 1), (3500, 512, 256, 1), (5000, 256, 512, 1), (3500, 256, 256, 1),
    (4096, 256, 256, 0), (7000, 128, 256, 0),          # dW's blocks would be wider, and it contracts over far more than dHidden
    (256, 64, 24000, 0),                               # dHidden's would be
])
def test_dhidden_and_dw_in_one_launch(N, H, V, together):
    i = _check(N, H, V, 1 << 14, 0, 0, N)
    assert i.rows == N and i.together == together


def test_bad_arguments_are_rejected():
    for a in [(0, 8, 8, 1, 0, 0, 0), (10, 8, 8, 1, 0, 5, 0), (10, 8, 8, 1, 0, 0, 11), (10, 8, 8, 1, 0, -1, 0),
              (10, 8, 8, 1, B.ALST_FLAG_FORWARD_ONLY, 0, 0), (10, 8, 8, 1, 1 << 20, 0, 0)]:
        with pytest.raises(B.AlstError):
            B.alst_debug_ce_chunk(*a)
