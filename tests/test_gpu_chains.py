"""Chains of blocks on persistent workgroups: contractions of an odd and an even number of k-steps (an odd one swaps the
LDS stages from block to block), of the least number of k-steps that a chain takes, several blocks per workgroup with a last
round in halves or none, and dense rows that end inside the chain's last row block.  That they run on chains is the library's
own choice (alst_debug_layer, alst_debug_ce_chunk).  Against the fp64 oracle, bar as in the other parity tests: 2e-2 of max |ref| per output."""
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


@pytest.mark.parametrize("name,N,H,V,n_valid", [
    # a chain from 1025 blocks on (the host's count of N rows)
    ("five_k_steps_and_halves", 1024, 320, 66000, 1000),                # 4 x 258 blocks
    ("four_k_steps", 1280, 256, 53000, 1280),                           # 5 x 208
    ("seven_k_steps_fewer_blocks_than_workgroups", 1300, 448, 45000, 200),
    ("six_k_steps_rows_end_in_the_first_half", 1100, 384, 54000, 300),
])
def test_logits(name, N, H, V, n_valid):
    wl = synth.custom(name, N, H, V, 1024, ignore_frac=0.0, seed=61)
    h, W, y = synth.make_inputs(wl)
    y[np.random.default_rng(62).choice(N, N - n_valid, replace=False)] = IGN
    assert all(i.logits_chained for i in G.ce_chunks(N, H, V, 1024, 0, n_valid))
    f, dH, dW = _oracle(h, W, y)
    r = G.run_fused(h, W, y, 1024)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    s = G.run_split(h, W, y, 1024)
    assert s.status_bwd == B.ALST_OK and s.loss_bits == r.loss_bits
    _check(s, f, dH, dW, name + " split", valid=(y != IGN))


@pytest.mark.parametrize("N,K,M", [
    (1000, 320, 33000),                # 4 x 129 blocks, ragged: halves behind chains of two
    (2048, 448, 17408),                # 8 x 68
    (1000, 1024, 24832),               # 4 x 97: chains of two, chains of one and padding numbers in between; no halves
    (1024, 1024, 24576),               # 256 + 128: as many halves as fit, nothing ragged
    (1153, 1024, 14400),               # 5 x 57, the last half has one row
    (1024, 320, 33536),                # 4 x 131: no halves, nothing ragged
])
def test_linear(N, K, M):
    assert B.alst_debug_layer(2, N, K, M, 4096).product_chained
    x, W, dy = TL._inputs(N, K, M, 63)
    got = TL._run(x, W, dy, 4096)
    for g, r in zip(got, (lorc.forward(x, W), *lorc.backward(x, W, dy))):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,H,I", [
    (1100, 320, 26400),                # 5 x 207 blocks of 5 k-steps, ragged, 11 of them in halves
    (1280, 256, 26624),                # 5 x 208, nothing ragged, halves
])
def test_gated(N, H, I):
    assert all(B.alst_debug_layer(op, N, H, I, 2048).gated_chained for op in (0, 1))
    wl = synth.MlpWorkload("odd", N, H, I, 2048, seed=64)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 2048)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL
