"""The rows per launch that layer calls work in (host arithmetic): the launches of a call never take more
rounds of the 256 compute units than one launch per tile of the caller would, whatever the extents, and the
chunks fit what the workspace holds."""
import math
import os
import random

import pytest

from paper_2506_13996_amd import binding as B

MLP_FORWARD, MLP_BACKWARD, LINEAR_FORWARD, LINEAR_DX = range(4)


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2506_13996_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def _launches(op, K, M):
    """(columns of output blocks, k-steps per block, last round in halves) of a chunk's launches."""
    up = lambda a, b: -(-a // b)
    t = K % 64 == 0 and M % 64 == 0
    return {MLP_FORWARD: [(up(M, 128), up(K, 64), True), (up(K, 256), up(M, 64), True)],
            MLP_BACKWARD: [(up(M, 256), up(K, 64), t), (up(M, 128), up(K, 64), True), (up(K, 256), up(2 * M, 64), t)],
            LINEAR_FORWARD: [(up(M, 256), up(K, 64), True)],
            LINEAR_DX: [(up(K, 256), up(M, 64), M % 64 == 0)]}[op]


def _rounds(blocks, halves):
    left = blocks % 256
    return blocks // 256 + (0 if left == 0 else 0.625 if halves and left <= 128 else 1)


def _time(op, N, K, M, chunk, launch=4):
    """Of a call in chunks of that many rows, in k-steps of one block: rounds times (k-steps + 4), and
    `launch` per launch."""
    per = lambda rows: sum(_rounds(-(-rows // 256) * cols, halves) * (k + 4) + launch
                           for cols, k, halves in _launches(op, K, M))
    return N // chunk * per(chunk) + (per(N % chunk) if N % chunk else 0)


# calls whose tiles were whole rounds of the compute units
@pytest.mark.parametrize("op,N,K,M,tile", [
    (LINEAR_FORWARD, 65536, 4096, 4096, 8192), (LINEAR_DX, 65536, 4096, 4096, 65536),
    (LINEAR_FORWARD, 16384, 4096, 16384, 8192), (LINEAR_FORWARD, 131072, 1024, 1024, 131072),
    (LINEAR_DX, 98304, 2048, 8192, 16384), (MLP_FORWARD, 32768, 2048, 8192, 8192),
    (MLP_FORWARD, 65536, 1024, 4096, 65536), (MLP_BACKWARD, 65536, 1024, 4096, 65536),
    (MLP_FORWARD, 32768, 4096, 11008, 32768), (MLP_BACKWARD, 32768, 2048, 8192, 8192),
])
def test_whole_rounds_stay_whole(op, N, K, M, tile):
    chunk = B.alst_debug_chunk_rows(op, N, K, M, tile)
    # (32768 x 4096 x 11008 forward: two chunks end in a round of halves each, 0.4 %)
    assert _time(op, N, K, M, chunk, launch=0) <= 1.005 * _time(op, N, K, M, tile, launch=0)


def test_no_call_takes_more_rounds_than_its_tiles_would():
    rng = random.Random(5)
    for _ in range(3000):
        op = rng.randrange(4)
        K, M = (8 * rng.randint(1, 700) if rng.random() < 0.3 else 256 * rng.randint(1, 64) for _ in range(2))
        N = int(2 ** rng.uniform(0, 19))
        tile = rng.choice([1, 100, 128, 300, 1024, 2048, 4096, 5000, 8192, 16384])
        chunk = B.alst_debug_chunk_rows(op, N, K, M, tile)
        assert chunk >= 256 and chunk % 256 == 0, (op, N, K, M, tile)
        if op == MLP_FORWARD:
            assert chunk <= -(-min(tile, N) // 256) * 256           # the workspace holds one tile
        # (3 %: the MLP's backward also weighs the number of its weight-gradient groups)
        assert _time(op, N, K, M, chunk) <= 1.03 * _time(op, N, K, M, min(tile, N)), (op, N, K, M, tile, chunk)


def test_bad_arguments_are_rejected():
    for a in [(4, 1, 8, 8, 1), (-1, 1, 8, 8, 1), (0, 0, 8, 8, 1), (0, 1, 8, (1 << 20) + 1, 1)]:
        with pytest.raises(B.AlstError):
            B.alst_debug_chunk_rows(*a)
