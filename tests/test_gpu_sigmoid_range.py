"""SwiGLU where the sigmoid is a subnormal number (gate between -88.7 and -87.3): silu, dg and du are normal numbers there
and reach the outputs, in every kernel that the gate and up projections run on.  Every row has one gate value g and one up
value u in all of I, dy and Wd select: y = I a, da = 1.  Bar: 2e-2 of max |ref| per output, as in the other parity
tests."""
import numpy as np
import pytest

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_mlp as TM

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("N,H,I,tile,columns,chained", [
    (192, 64, 128, 2048, 64, 0),       # small blocks
    (1032, 72, 1032, 2048, 0, 0),      # large blocks
    (4096, 256, 8448, 4096, 0, 1),     # chains of blocks: 16 x 66
])
def test_subnormal_sigmoid(N, H, I, tile, columns, chained):
    for op in (0, 1):
        i = B.alst_debug_layer(op, N, H, I, tile)
        assert (i.gated_columns, i.gated_chained) == (columns, chained)
    g = np.array([-87.5, -88.0, -88.5])[np.arange(N) % 3]
    u = 2.0 ** 20
    x, Wg, Wu = np.zeros((N, H)), np.zeros((I, H)), np.zeros((I, H))
    Wd, dy = np.zeros((H, I)), np.zeros((N, H))
    x[:, 0], x[:, 1], Wg[:, 0], Wu[:, 1] = g, 1.0, 1.0, u
    Wd[3], dy[:, 3] = 1.0, 1.0                         # da = 1; y = (0, 0, 0, sum of a, 0, ..)
    bits = [synth.f32_to_bf16_bits(t.astype(np.float32)) for t in (x, Wg, Wu, Wd, dy)]
    y, dx, (dWg, dWu, dWd) = TM._run(*bits, tile)

    sg = 1.0 / (1.0 + np.exp(-g))
    assert (sg > 0).all() and (sg < np.finfo(np.float32).tiny).all()
    silu = g * sg
    a, dg, du = silu * u, u * sg * (1.0 + g * (1.0 - sg)), silu
    ref_y, ref_dx = np.zeros((N, H)), np.zeros((N, H))
    ref_y[:, 3] = I * a
    ref_dx[:, 0], ref_dx[:, 1] = I * dg, I * du * u
    ref_dWg, ref_dWu, ref_dWd = np.zeros((I, H)), np.zeros((I, H)), np.zeros((H, I))
    ref_dWg[:, 0], ref_dWg[:, 1] = (dg * g).sum(), dg.sum()
    ref_dWu[:, 0], ref_dWu[:, 1] = (du * g).sum(), du.sum()
    ref_dWd[3] = a.sum()
    for name, got, ref in (("y", y, ref_y), ("dx", dx, ref_dx), ("dWg", dWg, ref_dWg), ("dWu", dWu, ref_dWu), ("dWd", dWd, ref_dWd)):
        assert G.grad_err(got, ref) <= TOL, name
