"""Launches in small blocks of 64 x 64 or 64 x 128: the counts at which they begin and end, extents that end inside a
block, contractions shorter and longer than the ring of stages, and ranges of k that leave a wavefront without steps; next to them, ragged launches just large enough for 256 x 256 blocks.  Against the fp64
oracle, bar as in the other parity tests: 2e-2 of max |ref| per output (bf16 rounding of intermediates and
outputs, 2^-9 relative each; the order of the fp32 sums is far below that)."""
import pytest

from oracle import tiled_linear_oracle as lorc
from oracle import tiled_mlp_oracle as morc
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_linear as TL
from tests import test_gpu_mlp as TM

pytestmark = pytest.mark.gpu
TOL = 2e-2


def small_columns(rows, cols):
    """Which blocks a product's launch takes: at most one round of 256 small ones."""
    r = -(-rows // 64)
    return 64 if r * -(-cols // 64) <= 256 else 128 if r * -(-cols // 128) <= 256 else 0


@pytest.mark.parametrize("N,K,M,forward,wgrad", [
    (1024, 8, 1024, 64, 64),           # 256 blocks of 64 x 64; one chunk of 8 k
    (1024, 72, 1032, 128, 64),         # one column of blocks more; a second k-step of 8
    (1000, 520, 1000, 64, 64),         # the ring's 8 stages filled once and a tail
    (1024, 648, 2048, 128, 128),       # 256 blocks of 64 x 128, more k-steps than their 5 stages
    (1025, 264, 2056, 0, 64),          # beyond: large blocks, ragged in every extent
    (65, 1096, 72, 64, 64),            # 18 k-steps forward; 65 rows of x are three steps of 32 k for four wavefronts
    (2056, 1288, 2056, 0, 0),          # large blocks in all three products
    (1, 8, 8, 64, 64),
])
def test_linear(N, K, M, forward, wgrad):
    assert small_columns(N, M) == forward and small_columns(K, M) == wgrad
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
])
def test_mlp(N, H, I, gated):
    assert small_columns(N, 2 * I) == gated
    wl = synth.MlpWorkload("small", N, H, I, 2048, seed=52)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 2048)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL
