"""The launch schedule of the tiled MLP and linear layer: chunks of rows that span several of the
caller's tiles, weight-gradient groups, da and a in one place, against the fp64 oracle.  Bar as in the
other parity tests of these layers: 2e-2 of max |ref| per output."""
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


@pytest.mark.parametrize("flags", [0, B.ALST_FLAG_DW_FP32, B.ALST_FLAG_DW_FP32 | B.ALST_FLAG_DW_ACCUMULATE])
@pytest.mark.parametrize("N,H,I,tile", [
    (4500, 64, 128, 128),       # backward: 2048 rows per chunk, the last one ragged; forward: 256
    (4500, 72, 136, 100),       # the weights as they are (not whole k-steps)
    (2049, 128, 192, 7),        # one row in the last chunk
    (2048, 256, 128, 256),      # exactly one chunk
])
def test_mlp_chunks(N, H, I, tile, flags):
    wl = synth.MlpWorkload("chunks", N, H, I, tile, seed=21)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    init = None
    if flags & B.ALST_FLAG_DW_ACCUMULATE:
        init = [torch.full(s, 0.25, device="cuda") for s in ((I, H), (I, H), (H, I))]
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, tile, flags=flags, init=init)
    if init:
        gW = [g - 0.25 for g in gW]
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    for g, r in zip((y, dx, *gW), ref):
        assert G.grad_err(g, r) <= TOL


@pytest.mark.parametrize("N,K,M,tile", [
    (16385, 64, 72, 128),       # one row in the second weight-gradient group
    (66000, 8, 16, 300),        # 220 tiles in one launch of y and of dx
    (17000, 16, 64, 16640),     # a tile longer than a group
])
def test_linear_chunks(N, K, M, tile):
    x, W, dy = TL._inputs(N, K, M, 22)
    got = TL._run(x, W, dy, tile)
    for g, r in zip(got, (lorc.forward(x, W), *lorc.backward(x, W, dy))):
        assert G.grad_err(g, r) <= TOL


def test_several_launches_of_y_and_dx():
    """Rows of more than 128 MB of either operand: y and dx in several launches, the last of them short.  Rows on
    both sides of every seam and a sample of the others against float64 on the same device."""
    N, K, M = 33_000, 4104, 2184
    chunks = [B.alst_debug_chunk_rows(op, N, K, M, 4096) for op in (2, 3)]
    assert all(N // 3 < c < N for c in chunks)
    g = torch.Generator(device="cuda").manual_seed(24)
    x, W, dy = (torch.randn(s, device="cuda", generator=g).to(torch.bfloat16) for s in ((N, K), (M, K), (N, M)))
    y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    dW = torch.empty_like(W)
    B.alst_tiled_linear_forward(x, W, 4096, y=y)
    ws = torch.empty(B.alst_tiled_linear_workspace_bytes(N, K, M, 4096, True), dtype=torch.uint8, device="cuda")
    B.alst_tiled_linear_backward(x, W, dy, 4096, dx=dx, dW=dW, workspace=ws)
    assert torch.isfinite(y).all() and torch.isfinite(dx).all()
    seams = [r for c in chunks for at in range(c, N, c) for r in (at - 2, at - 1, at, at + 1)]
    rows = torch.tensor(sorted({0, 1, N - 2, N - 1, *seams, *range(7, N, 997)}), device="cuda")
    for got, ref in ((y, x[rows].double() @ W.double().t()), (dx, dy[rows].double() @ W.double())):
        assert float((got[rows].double() - ref).abs().max() / ref.abs().max()) <= TOL


def test_tile_size_does_not_reach_rows():
    """y and dx of a row are the same bits whatever the caller's tile."""
    wl = synth.MlpWorkload("t", 1500, 128, 256, 0, seed=23)
    inputs = synth.make_mlp_inputs(wl)
    outs = [TM._run(*inputs, tile) for tile in (1500, 512, 100)]
    for y, dx, _ in outs[1:]:
        assert np.array_equal(y, outs[0][0]) and np.array_equal(dx, outs[0][1])
