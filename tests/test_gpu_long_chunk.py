"""A chunk of more than 4096 row blocks (a tile beyond 1048576 rows) whose valid rows are few: its full
extent has blocks enough for every compute unit and is never cut, while the rows that take part are few
enough for dHidden's contraction over the vocabulary to be cut into ranges.  The results of the valid rows
against the oracle on those rows (rows are independent), exact zeros everywhere else."""
import numpy as np
import pytest
import torch

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


def test_as_many_rows_as_a_grid_of_one_workgroup_per_row_holds():
    """A grid has fewer than 2^32 threads, so a chunk must not be so long that its gather (one workgroup of
    256 per row and those that zero the ignored rows of dHidden) does not fit: here 2^24 - 256 rows, in one
    tile."""
    N, H, V, n_valid = 16_776_960, 8, 40, 700
    g = torch.Generator(device="cuda").manual_seed(83)
    hd = torch.randn((N, H), device="cuda", generator=g).to(torch.bfloat16)
    Wd = torch.randn((V, H), device="cuda", generator=g).mul_(0.02).to(torch.bfloat16)
    rows = np.sort(np.random.default_rng(84).choice(N, n_valid, replace=False))
    y = np.full(N, IGN, dtype=np.int32)
    y[rows] = np.random.default_rng(85).integers(0, V, n_valid)
    at = torch.from_numpy(rows).cuda()
    ws = B.alloc_workspace(N, H, V, N)
    loss, dH = torch.zeros(1, device="cuda"), torch.full((N, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    dW = torch.empty((V, H), dtype=torch.bfloat16, device="cuda")
    B.alst_tiled_ce_forward_backward(hd, Wd, torch.from_numpy(y).cuda(), N, IGN, 1.0, loss_out=loss, dHidden=dH,
                                     dW=dW, workspace=ws)
    assert B.alst_last_device_status(ws) == B.ALST_OK
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
    f, ref_dH, ref_dW = _oracle(bits(hd[at]), bits(Wd), y[rows])
    assert abs(float(loss.item()) - f["loss"]) <= LOSS_RTOL * abs(f["loss"])
    assert G.grad_err(G.bf16_dev_to_f64(dH[at]), ref_dH) <= GRAD_TOL
    assert G.grad_err(G.bf16_dev_to_f64(dW), ref_dW) <= GRAD_TOL
    dH[at] = 0
    assert int(torch.count_nonzero(dH.view(torch.int16))) == 0
