"""Launches whose last round of output blocks is worked on in halves of 128 rows: whole rounds in front of
it and none, halves without rows, extents that end inside a half (behind chains of blocks: test_gpu_chains.py),
against the fp64 oracle.  Launches of few blocks, which run on smaller ones, are next to them.  Bar as in the other parity tests: 2e-2 of max |ref| per output."""
import numpy as np
import pytest

from oracle import tiled_linear_oracle as lorc
from oracle import tiled_mlp_oracle as morc
from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_linear as TL
from tests import test_gpu_mlp as TM
from tests.test_gpu_parity import IGN, _check, _oracle

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("N,K,M", [
    (1024, 384, 24576),         # 256 + 128 blocks: as many halves as fit
    (1024, 320, 24584),         # 256 + 132: none
    (800, 256, 24200),          # 256 + 124, the second halves of the last rows are empty
    (900, 72, 24320),           # the last half has 4 rows; K is not whole k-steps
    (1153, 320, 14400),         # 256 + 29, the last half has one row
    (129, 64, 256),             # (small blocks)
    (128, 512, 264),
])
def test_linear(N, K, M):
    i = B.alst_debug_layer(2, N, K, M, 1024)
    assert not i.product_chained and (i.product_columns == 0) == (M > 1000)
    x, W, dy = TL._inputs(N, K, M, 31)
    got = TL._run(x, W, dy, 1024)
    for g, r in zip(got, (lorc.forward(x, W), *lorc.backward(x, W, dy))):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,H,I", [
    (1024, 256, 12288),         # gate / up: 256 + 128 blocks
    (900, 320, 12168),          # rows and columns ragged
    (140, 256, 640),            # (small blocks)
])
def test_mlp(N, H, I):
    i = B.alst_debug_layer(1, N, H, I, 1024)
    assert not i.gated_chained and (i.gated_columns == 0) == (I > 1000)
    wl = synth.MlpWorkload("halves", N, H, I, 1024, seed=32)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 1024)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("name,N,H,V,n_valid,left,empty_half", [
    # left: output blocks of the logits in the last round; empty_half: its last row block's second half has no row
    ("whole_rounds_then_halves", 1024, 64, 24576, 1024, 128, False),
    ("ragged", 1000, 72, 24300, 950, 124, False),
    ("more_than_halves_take", 600, 64, 33000, 517, 131, True),
    ("second_half_without_rows", 600, 64, 33000, 350, 2, True),
    ("a_last_half_with_one_row", 1153, 64, 14800, 1153, 34, False),
    ("small_blocks", 129, 64, 300, 129, 2, False),
])
def test_cross_entropy(name, N, H, V, n_valid, left, empty_half):
    row_blocks, columns = -(-n_valid // 256), -(-V // 256)
    i = B.alst_debug_ce_chunk(N, H, V, 1024, 0, 0, n_valid)
    assert i.rows == N and not i.logits_chained and (i.logits_columns == 0) == (name != "small_blocks")
    assert row_blocks * columns % 256 == left and ((n_valid - 1) % 256 < 128) == empty_half
    wl = synth.custom(name, N, H, V, 1024, ignore_frac=0.0, seed=33)
    h, W, y = synth.make_inputs(wl)
    y[np.random.default_rng(34).choice(N, N - n_valid, replace=False)] = IGN
    f, dH, dW = _oracle(h, W, y)
    r = G.run_fused(h, W, y, 1024)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    s = G.run_split(h, W, y, 1024)
    assert s.status_bwd == B.ALST_OK and s.loss_bits == r.loss_bits
    _check(s, f, dH, dW, name + " split", valid=(y != IGN))
    assert (s.lse.view(np.uint32) == r.lse.view(np.uint32)).all()
