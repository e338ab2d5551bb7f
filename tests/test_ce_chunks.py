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


def test_bad_arguments_are_rejected():
    for a in [(0, 8, 8, 1, 0, 0, 0), (10, 8, 8, 1, 0, 5, 0), (10, 8, 8, 1, 0, 0, 11), (10, 8, 8, 1, 0, -1, 0),
              (10, 8, 8, 1, B.ALST_FLAG_FORWARD_ONLY, 0, 0), (10, 8, 8, 1, 1 << 20, 0, 0)]:
        with pytest.raises(B.AlstError):
            B.alst_debug_ce_chunk(*a)
