"""Launches in small blocks of 64 x 64 or 64 x 128: the counts at which they begin and end, extents that end inside a
block, contractions shorter and longer than the ring of stages, ranges of k that leave a wavefront without steps, and
row numbering inside the gather launch; next to them, ragged launches just large enough for 256 x 256 blocks.  Which blocks a
case runs on is the library's own choice (alst_debug_layer, alst_debug_ce_chunk).  Against the fp64 oracle, bar as in the other parity tests: 2e-2 of max |ref| per output (bf16 rounding of intermediates and
outputs, 2^-9 relative each; the order of the fp32 sums is far below that)."""
import numpy as np
import pytest

from oracle import tiled_ce_oracle as orc
from oracle import tiled_linear_oracle as lorc
from oracle import tiled_mlp_oracle as morc
from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_linear as TL
from tests import test_gpu_mlp as TM
from tests.test_gpu_parity import IGN, _check, _oracle, _redo_case

pytestmark = pytest.mark.gpu
TOL = 2e-2


MLP_FORWARD, MLP_BACKWARD, LINEAR_FORWARD, LINEAR_BACKWARD = range(4)


def gradients(op, N, K, M, tile):
    """Columns of the blocks of dx and of the weight gradients (0: 256 x 256 blocks), whether they are one launch."""
    i = B.alst_debug_layer(op, N, K, M, tile)
    assert i.rows == N                 # (one chunk)
    return i.product_columns, i.wgrad_columns, i.together


@pytest.mark.parametrize("N,K,M,forward,backward", [
    (1024, 8, 1024, 64, (64, 64, 1)),          # 256 blocks of 64 x 64; one chunk of 8 k
    (1024, 72, 1032, 128, (64, 64, 1)),        # one column of blocks more; a second k-step of 8
    (1000, 520, 1000, 64, (128, 128, 1)),      # the ring's 8 stages filled once and a tail
    (1024, 648, 2048, 128, (64, 128, 0)),      # 256 blocks of 64 x 128, more k-steps than their 5 stages
    (1025, 264, 2056, 0, (64, 64, 1)),         # beyond: large blocks, ragged in every extent
    (65, 1096, 72, 64, (64, 64, 1)),           # 18 k-steps forward; 65 rows of x are three steps of 32 k for four wavefronts
    (2056, 1288, 2056, 0, (0, 0, 0)),          # large blocks in all three products
    (1, 8, 8, 64, (64, 64, 1)),
    (520, 2056, 2048, 128, (128, 0, 0)),
    (200, 2048, 1032, 64, (64, 0, 0)),
    (1500, 1024, 2048, 0, (128, 128, 0)),
])
def test_linear(N, K, M, forward, backward):
    assert B.alst_debug_layer(LINEAR_FORWARD, N, K, M, 4096).product_columns == forward
    assert gradients(LINEAR_BACKWARD, N, K, M, 4096) == backward
    x, W, dy = TL._inputs(N, K, M, 51)
    got = TL._run(x, W, dy, 4096)
    for g, r in zip(got, (lorc.forward(x, W), *lorc.backward(x, W, dy))):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,H,I,gated", [
    (512, 256, 1000, 64),              # the last block has 8 of its 32 columns of I: lanes that store nothing
    (1000, 264, 512, 64),              # the last rows end inside a wavefront's 16
    (300, 64, 1720, 128),
    (1000, 320, 1000, 128),
    (1032, 72, 1032, 0),               # large blocks
    (500, 320, 448, 64),               # whole k-steps: da is made in the gated launch
    (1000, 256, 832, 128),
    (1000, 1024, 832, 128),            # 16 k-steps: every stage of the rings of da and of g and u is used
    (500, 1096, 448, 64),
])
def test_mlp(N, H, I, gated):
    assert [B.alst_debug_layer(op, N, H, I, 2048).gated_columns for op in (MLP_FORWARD, MLP_BACKWARD)] == [gated] * 2
    wl = synth.MlpWorkload("small", N, H, I, 2048, seed=52)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 2048)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL


# route: columns of the small blocks of the last chunk's logits, dHidden and dW (0: 256 x 256), whether dHidden and dW are one
# launch, whether the gather launch numbers the rows
@pytest.mark.parametrize("name,N,H,V,tile,n_valid,route", [
    ("gather_numbers_1024_rows", 1024, 256, 2048, 1024, 1000, (128, 128, 128, 1, 1)),        # logits: 256 blocks of 64 x 128
    ("one_row_more", 1025, 256, 2048, 2048, 1000, (0, 128, 128, 1, 0)),      # a launch of its own numbers the rows
    ("every_row_valid", 1024, 72, 500, 1024, 1024, (128, 64, 64, 1, 1)),
    ("no_row_valid", 700, 64, 300, 1024, 0, (128, 64, 64, 1, 1)),
    ("one_row_valid", 64, 64, 300, 64, 1, (128, 64, 64, 1, 1)),
    ("two_chunks", 1000, 64, 3000, 128, 900, (128, 64, 64, 1, 0)),           # dense rows beyond one chunk
    ("large_logits_small_gradients", 1000, 136, 6000, 1024, 960, (0, 128, 128, 0, 1)),
    ("small_logits_large_dw", 128, 2304, 2304, 128, 120, (128, 128, 0, 0, 1)),
    ("vocabulary_ends_before_the_last_small_block", 200, 64, 4097, 256, 200, (128, 64, 64, 1, 1)),
    ("dHidden_64_dW_128_apart", 200, 512, 4000, 256, 190, (128, 64, 128, 0, 1)),
    ("dHidden_128_dW_64_apart", 1024, 512, 2048, 1024, 900, (128, 128, 64, 0, 1)),
    ("large_dHidden_dW_64", 3000, 256, 1500, 4096, 2900, (0, 0, 64, 0, 0)),
])
def test_cross_entropy(name, N, H, V, tile, n_valid, route):
    i = G.ce_chunks(N, H, V, tile, 0, n_valid)[-1]
    assert (i.logits_columns, i.dhidden_columns, i.dw_columns, i.together, i.numbered_by_gather) == route
    wl = synth.custom(name, N, H, V, tile, ignore_frac=0.0, seed=53)
    h, W, y = synth.make_inputs(wl)
    y[np.random.default_rng(54).choice(N, N - n_valid, replace=False)] = IGN
    r = G.run_fused(h, W, y, tile)
    assert r.n_valid == n_valid and r.status == B.ALST_OK
    if n_valid == 0:
        assert r.loss == 0.0 and not r.dH.any() and not r.dW.any() and not r.lse.any()
        return
    f, dH, dW = _oracle(h, W, y)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    s = G.run_split(h, W, y, tile)
    assert s.status_bwd == B.ALST_OK and s.loss_bits == r.loss_bits
    _check(s, f, dH, dW, name + " split", valid=(y != IGN))


@pytest.mark.parametrize("N,K,M,joint", [
    (512, 512, 1536, 64),              # 64 blocks of dx and 192 of dW: one round
    (520, 512, 1536, 128),             # a row of blocks more
    (1000, 1000, 904, 128),            # ragged in every extent; one round, 15 k-steps
    (4000, 256, 256, 0),               # one round of 64 x 128, but dW's contraction is too long for blocks of twice the width
    (1024, 1024, 2048, 0),             # 128 + 256 blocks of 64 x 128: two launches, both small: 64 x 64 and 64 x 128
    (5, 8, 16, 64),
])
def test_linear_backward_in_one_launch(N, K, M, joint):
    assert gradients(LINEAR_BACKWARD, N, K, M, 4096) == ((joint, joint, 1) if joint else (64, 64 if N == 4000 else 128, 0))
    x, W, dy = TL._inputs(N, K, M, 58)
    got = TL._run(x, W, dy, 4096)
    for g, r in zip(got, (lorc.forward(x, W), *lorc.backward(x, W, dy))):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,H,I,joint", [
    (512, 256, 1024, 64),              # 32 blocks of dx and 3 x 64 of the weights' gradients
    (1000, 256, 1024, 64),             # 64: one round
    (1032, 256, 1024, 128),
    (300, 520, 1000, 128),             # ragged: transposed weights lie where the sums would
    (256, 128, 4096, 0),               # the same for dx
    (600, 384, 2048, 0),
])
def test_mlp_backward_in_one_launch(N, H, I, joint):
    assert gradients(MLP_BACKWARD, N, H, I, 2048) == ((joint, joint, 1) if joint else (64, 128 if H == 128 else 0, 0))
    wl = synth.MlpWorkload("joint", N, H, I, 2048, seed=59)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 2048)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("name,N,H,V,tile,n_valid,route", [
    ("one_round_of_both", 512, 256, 4096, 512, 486, (128, 128, 128, 1, 1)),
    ("fewer_rows_than_the_chunk", 512, 256, 4096, 512, 100, (128, 128, 128, 1, 1)),
    ("no_row_valid", 512, 256, 4096, 512, 0, (128, 128, 128, 1, 1)),
    ("last_chunk_without_rows", 1000, 64, 3000, 128, 120, (128, 64, 64, 1, 0)),
    ("two_launches", 512, 512, 4096, 512, 486, (128, 128, 128, 0, 1)),
    ("wider_blocks_would_cost_more", 4096, 256, 256, 4096, 4000, (128, 64, 64, 0, 0)),
])
def test_cross_entropy_gradients_in_one_launch(name, N, H, V, tile, n_valid, route):
    test_cross_entropy(name, N, H, V, tile, n_valid, route)


def test_a_label_out_of_range_is_reported_where_the_gather_numbers_the_rows():
    wl = synth.custom("bad", 300, 64, 500, 512, ignore_frac=0.1, seed=55)
    h, W, y = synth.make_inputs(wl)
    ok = y.copy()
    ok[137] = IGN
    y[137] = 500
    r = G.run_fused(h, W, y, 512)
    assert r.status == B.ALST_ERR_LABEL_RANGE and r.n_valid == int((ok != IGN).sum())
    f, dH, dW = _oracle(h, W, ok)
    r.status = B.ALST_OK
    _check(r, f, dH, dW, "label out of range", valid=(ok != IGN))


def test_second_pass_in_large_blocks():
    """The second logits pass for some rows of a chunk, at a size beyond the small blocks."""
    N, H, V = 640, 64, 6000
    assert B.alst_debug_ce_chunk(N, H, V, 1024, 0, 0, N).logits_columns == 0
    wl = synth.custom("redo", N, H, V, 1024, ignore_frac=0.1, seed=56)
    h, _, y = synth.make_inputs(wl)
    W = synth.normal_bf16(V, H, 0.2, 57, synth.STREAM_W)
    hm = orc.bf16_bits_to_f64(h).copy()
    hm[::3] *= 40.0
    f = _redo_case("mixed, large blocks", synth.f32_to_bf16_bits(hm.astype(np.float32)), W, y, 1024)
    assert (np.abs(f["lse"]) > 90.0)[::3][(y != IGN)[::3]].all()
