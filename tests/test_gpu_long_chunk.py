"""A chunk of more than 4096 row blocks (a tile beyond 1048576 rows) whose valid rows are few: its full
extent has blocks enough for every compute unit and is never cut, while the rows that take part are few
enough for dHidden's contraction over the vocabulary to be cut into ranges.  The results of the valid rows
against the oracle on those rows (rows are independent), exact zeros everywhere else."""
import numpy as np
import pytest

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import GRAD_TOL, IGN, LOSS_RTOL, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,n_valid", [(1024, 500), (2048, 8000)])
def test_few_valid_rows_in_a_long_chunk(V, n_valid):
    N, H = 1_048_832, 8
    h, W, y = synth.make_inputs(synth.custom("long_chunk", N, H, V, N, ignore_frac=0.0, seed=81))
    valid = np.zeros(N, dtype=bool)
    valid[np.random.default_rng(82).choice(N, n_valid, replace=False)] = True
    y = np.where(valid, y, IGN).astype(np.int32)
    f, dH, dW = _oracle(h[valid], W, y[valid])
    r = G.run_fused(h, W, y, N)                    # (fills dHidden with NaN beforehand)
    assert r.status == B.ALST_OK and r.n_valid == n_valid
    assert abs(r.loss - f["loss"]) <= LOSS_RTOL * abs(f["loss"])
    assert (r.dH[~valid] == 0.0).all()
    assert np.isfinite(r.dH[valid]).all(), "rows of dHidden that nothing has written"
    assert G.grad_err(r.dH[valid], dH) <= GRAD_TOL and G.grad_err(r.dW, dW) <= GRAD_TOL
