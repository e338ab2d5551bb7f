"""What the launches of a layer call run on (host arithmetic, the functions that the calls use): small blocks are at most one
round of the compute units and as narrow as that allows, whole k-steps only are chained, weights are read as they are only
where no room is left to transpose them."""
import os
import random

import pytest

from paper_2506_13996_amd import binding as B

MLP_FORWARD, MLP_BACKWARD, LINEAR_FORWARD, LINEAR_BACKWARD = range(4)
FP32, ADD = B.ALST_FLAG_DW_FP32, B.ALST_FLAG_DW_ACCUMULATE


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2506_13996_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def _blocks(columns, *products):
    return sum(-(-r // 64) * -(-c // columns) for r, c in products)


def _narrowest(*products):
    return next((c for c in (64, 128) if _blocks(c, *products) <= 256), 0)


def _check(op, N, K, M, tile, flags):
    i = B.alst_debug_layer(op, N, K, M, tile, flags)
    case = (op, N, K, M, tile, flags, [(n, getattr(i, n)) for n, _ in i._fields_])
    assert 1 <= i.rows <= N, case
    if op < LINEAR_FORWARD:
        assert i.gated_columns == _narrowest((i.rows, 2 * M)), case
        assert not (i.gated_columns and i.gated_chained), case
        assert not i.gated_chained or (K % 64 == 0 and K >= 256), case
    d = (i.rows, {MLP_FORWARD: K, MLP_BACKWARD: K, LINEAR_FORWARD: M, LINEAR_BACKWARD: K}[op])
    contraction = {MLP_FORWARD: M, MLP_BACKWARD: 2 * M, LINEAR_FORWARD: K, LINEAR_BACKWARD: M}[op]
    assert not i.product_chained or (i.product_columns == 0 and contraction % 64 == 0 and contraction >= 256), case
    if op in (MLP_FORWARD, LINEAR_FORWARD):
        assert i.product_columns == _narrowest(d) and not i.together, case
        return i
    weights = [(K, M)] * 2 + [(M, K)] if op == MLP_BACKWARD else [(K, M)]
    if i.together:
        assert i.transposed and i.product_columns == i.wgrad_columns and _blocks(i.wgrad_columns, d, *weights) <= 256, case
    else:
        assert i.product_columns == (_narrowest(d) if i.transposed else 0) and i.wgrad_columns == _narrowest(*weights), case
    whole = M % 64 == 0 and (K % 64 == 0 or op == LINEAR_BACKWARD)
    assert i.transposed or not whole, case
    if flags == FP32 and not whole:                    # (the sums lie in the outputs)
        assert not i.transposed, case
    return i


def test_random_shapes():
    rng = random.Random(5)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    seen = {op: set() for op in range(4)}
    for _ in range(6000):
        op = rng.randrange(4)
        step = rng.choice([8, 64])
        K, M = (max(step, log(8, 8192) // step * step) for _ in range(2))
        i = _check(op, log(1, 300_000), K, M, log(1, 1 << 17), rng.choice([0, 0, FP32, ADD, FP32 | ADD]))
        seen[op].add((i.gated_columns, i.gated_chained, i.product_columns, i.product_chained, i.wgrad_columns, i.together))
    assert all(len(s) >= 4 for s in seen.values()), seen


@pytest.mark.parametrize("op,N,K,M,tile,flags,transposed", [
    (LINEAR_BACKWARD, 300, 72, 136, 4096, 0, 1), (LINEAR_BACKWARD, 300, 72, 136, 4096, FP32, 0),
    (LINEAR_BACKWARD, 300, 72, 136, 4096, FP32 | ADD, 1), (LINEAR_BACKWARD, 16384, 72, 136, 256, 0, 1),
    (LINEAR_BACKWARD, 16385, 72, 136, 256, 0, 0), (LINEAR_BACKWARD, 16385, 72, 136, 20000, 0, 1),
    (LINEAR_BACKWARD, 16385, 72, 128, 256, FP32, 1), (MLP_BACKWARD, 300, 72, 136, 4096, 0, 1),
    (MLP_BACKWARD, 300, 72, 136, 4096, FP32, 0), (MLP_BACKWARD, 2400, 72, 136, 256, 0, 0), (MLP_BACKWARD, 2400, 64, 128, 256, FP32, 1),
])
def test_weights_transposed_or_as_they_are(op, N, K, M, tile, flags, transposed):
    assert _check(op, N, K, M, tile, flags).transposed == transposed


@pytest.mark.parametrize("op,N,K,M,together", [
    # one round of small blocks in all, as wide as each kind's alone
    (LINEAR_BACKWARD, 3800, 256, 256, 1), (MLP_BACKWARD, 2000, 256, 512, 1),
    # wider ones for the weight gradients: unless their contraction (N) is far longer than that of dx
    (LINEAR_BACKWARD, 512, 1024, 1024, 1), (LINEAR_BACKWARD, 5000, 256, 1024, 1), (LINEAR_BACKWARD, 4000, 256, 256, 0),
    (LINEAR_BACKWARD, 7900, 256, 256, 0), (LINEAR_BACKWARD, 14000, 128, 256, 0), (MLP_BACKWARD, 6000, 256, 512, 1),
    (MLP_BACKWARD, 7000, 256, 256, 0), (MLP_BACKWARD, 12000, 128, 256, 0),
    # wider ones for dx
    (LINEAR_BACKWARD, 2000, 256, 3072, 1), (LINEAR_BACKWARD, 300, 512, 2560, 0), (LINEAR_BACKWARD, 500, 128, 8192, 0),
    (MLP_BACKWARD, 400, 256, 1400, 1), (MLP_BACKWARD, 256, 128, 4096, 0),
])
def test_dx_and_weight_gradients_in_one_launch(op, N, K, M, together):
    i = _check(op, N, K, M, 1 << 16, 0)
    assert i.rows == N and i.together == together


def test_bad_arguments_are_rejected():
    for a in [(4, 8, 8, 8, 1), (-1, 8, 8, 8, 1), (0, 0, 8, 8, 1), (1, 8, 12, 8, 1), (2, 8, 8, 9, 1), (3, 8, 8, 8, 0),
              (3, 8, 8, 8, 1, B.ALST_FLAG_TILE_SCRATCH)]:
        with pytest.raises(B.AlstError):
            B.alst_debug_layer(*a)
