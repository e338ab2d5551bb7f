"""Weights whose extents are not whole k-steps: transposed into the room of the sums (calls of one group), read as they
are (several groups; fp32 overwrite outputs, which hold the sums), with what the sums' room is for done too (+=).
Against the fp64 oracle.  Bars: bf16 outputs 2e-2 of max |ref|, fp32 weight gradients 5e-3 (bf16 operands)."""
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
FP32, ADD = B.ALST_FLAG_DW_FP32, B.ALST_FLAG_DW_ACCUMULATE


def _init(shapes, top, flags):
    g = torch.Generator().manual_seed(5)
    dtype = torch.float32 if flags & FP32 else torch.bfloat16
    return [(torch.randn(s, generator=g).clamp_(-4, 4) * t).to(dtype).cuda() for s, t in zip(shapes, top)]


def _bar(flags):
    return 5e-3 if flags & FP32 else 2e-2


@pytest.mark.parametrize("flags", [0, ADD, FP32, FP32 | ADD])
@pytest.mark.parametrize("N,K,M,tile", [
    (300, 72, 136, 4096),
    (700, 264, 520, 128),
    (16500, 72, 136, 256),       # two groups
])
def test_linear(N, K, M, tile, flags):
    x, W, dy = TL._inputs(N, K, M, 71)
    ref = (lorc.forward(x, W), *lorc.backward(x, W, dy))
    init = _init([(M, K)], [float(np.abs(ref[2]).max())], flags)[0] if flags & ADD else None
    y, dx, dW = TL._run(x, W, dy, tile, flags=flags, init=init)
    assert G.grad_err(y, ref[0]) <= 2e-2 and G.grad_err(dx, ref[1]) <= 2e-2
    base = init.float().cpu().numpy().astype(np.float64) if flags & ADD else 0.0
    assert np.abs(dW - (base + ref[2])).max() / np.abs(ref[2]).max() <= _bar(flags)


@pytest.mark.parametrize("flags", [0, FP32, FP32 | ADD])
@pytest.mark.parametrize("N,H,I,tile", [
    (300, 72, 136, 4096),
    (257, 128, 200, 128),        # H is whole k-steps, I is not: Wu transposed begins inside one
    (2400, 72, 136, 256),        # two groups
])
def test_mlp(N, H, I, tile, flags):
    wl = synth.MlpWorkload("ragged", N, H, I, tile, seed=72)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    ref = (morc.forward(x, Wg, Wu, Wd, row_block=256), *morc.backward(x, Wg, Wu, Wd, dy, row_block=256))
    top = [float(np.abs(r).max()) for r in ref[2:]]
    init = _init([(I, H), (I, H), (H, I)], top, flags) if flags & ADD else None
    y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, tile, flags=flags, init=init)
    assert G.grad_err(y, ref[0]) <= 2e-2 and G.grad_err(dx, ref[1]) <= 2e-2
    for k, (g, r) in enumerate(zip(gW, ref[2:])):
        base = init[k].float().cpu().numpy().astype(np.float64) if flags & ADD else 0.0
        # (through a, dg, du, which are bf16: as the bf16 outputs)
        assert np.abs(g - (base + r)).max() / top[k] <= 2e-2
