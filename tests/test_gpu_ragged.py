"""Extents that end inside a block or a k-step, for every product of the tiled linear layer and MLP:
N, K (H) and M (I) at and next to multiples of 64 and 256, contractions of 1 to 5 k-steps.

The oracle is fp64.  Bar: 2e-2 of max |ref| per output, as in the other parity tests (bf16 rounding of
intermediates and outputs, 2^-9 relative each; observed about 3e-3)."""
import numpy as np
import pytest
import torch

from oracle import tiled_linear_oracle as lorc
from oracle import tiled_mlp_oracle as morc
from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_linear as TL
from tests import test_gpu_mlp as TM

pytestmark = pytest.mark.gpu
TOL = 2e-2

SHAPES = [
    # N, K, M, tile
    (1, 8, 8, 1),
    (63, 72, 264, 4096),
    (65, 128, 248, 64),
    (257, 136, 64, 128),
    (255, 192, 328, 300),
    (129, 200, 520, 100),
    (321, 264, 136, 256),
    (513, 256, 776, 200),         # whole k-steps, rows and columns ragged
    (1025, 320, 512, 512),
]


@pytest.mark.parametrize("N,K,M,tile", SHAPES)
def test_linear_ragged(N, K, M, tile):
    x, W, dy = TL._inputs(N, K, M, 11)
    got = TL._run(x, W, dy, tile)
    ref = (lorc.forward(x, W), *lorc.backward(x, W, dy))
    for g, r in zip(got, ref):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,H,I,tile", SHAPES)
def test_mlp_ragged(N, H, I, tile):
    wl = synth.MlpWorkload("ragged", N, H, I, tile, seed=12)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, tile)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL


def test_infinity_in_the_last_row_stays_there():
    """The last row of x is what a block reads in place of the rows it lacks, and the last k-row of dW's
    contraction: an infinity in it reaches its own outputs only."""
    N, K, M = 70, 72, 136
    x, W, dy = TL._inputs(N, K, M, 13)
    ref_y, (ref_dx, ref_dW) = lorc.forward(x, W), lorc.backward(x, W, dy)
    x = x.copy()
    x[-1, 3] = 0x7f80                                   # +inf
    y, dx, dW = TL._run(x, W, dy, 64)
    assert G.grad_err(y[:-1], ref_y[:-1]) <= TOL and np.isinf(y[-1]).all()
    assert G.grad_err(dx, ref_dx) <= TOL
    others = np.arange(K) != 3
    ref_dW[:, 3] = 0.0
    assert np.isinf(dW[:, 3]).all()
    got = dW[:, others]
    assert G.grad_err(got, ref_dW[:, others]) <= TOL          # (x differs nowhere else)
