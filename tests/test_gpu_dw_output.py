"""The weight gradient in every output form (bf16 / fp32, overwrite / accumulate) when it is complete in one
launch, when it is the sum of several, when the launches behind the last dense row are empty, and when
there is no dense row at all; H and V end inside a block.

Bars: fp32 output 5e-3 of max |dW| (bf16 operands, as test_gpu_linear), bf16 output 2e-2."""
import numpy as np
import pytest
import torch

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import IGN, _oracle

pytestmark = pytest.mark.gpu

FORMS = [0, B.ALST_FLAG_DW_FP32, B.ALST_FLAG_DW_ACCUMULATE, B.ALST_FLAG_DW_FP32 | B.ALST_FLAG_DW_ACCUMULATE]


@pytest.mark.parametrize("flags", FORMS)
@pytest.mark.parametrize("name,N,H,V,tile,ignored,groups", [
    # groups: dW groups (of one tile rounded up to 256) with dense rows, of all
    ("one_group", 200, 72, 520, 100, 0, (1, 1)),
    ("two_groups", 300, 72, 520, 100, 0, (2, 2)),
    ("three_groups", 700, 264, 328, 256, 0, (3, 3)),
    ("five_groups", 1200, 264, 328, 256, 0, (5, 5)),
    ("dense_rows_end_in_the_second_group", 1200, 72, 264, 256, 700, (2, 5)),
    ("no_dense_row", 600, 72, 264, 256, 600, (0, 3)),
])
def test_dw_forms(name, N, H, V, tile, ignored, groups, flags):
    chunks = G.ce_chunks(N, H, V, tile, flags | B.ALST_FLAG_TILE_SCRATCH, N - ignored)
    assert groups == (len({c.group0 for c in chunks if c.first < N - ignored}), len({c.group0 for c in chunks}))
    wl = synth.custom(name, N, H, V, tile, ignore_frac=0.0, seed=62)
    h, W, y = synth.make_inputs(wl)
    y = y.copy()
    y[:ignored] = IGN
    ref = _oracle(h, W, y)[2] if ignored < N else np.zeros((V, H))
    top = np.abs(ref).max() or 1.0
    dtype = torch.float32 if flags & B.ALST_FLAG_DW_FP32 else torch.bfloat16
    init = (torch.randn((V, H), generator=torch.Generator().manual_seed(1)).clamp_(-4, 4) * float(top)).to(dtype).cuda()
    r = G.run_fused(h, W, y, tile, flags=flags | B.ALST_FLAG_TILE_SCRATCH,      # (a group is one tile)
                    dW_init=init if flags & B.ALST_FLAG_DW_ACCUMULATE else None)
    base = init.float().cpu().numpy().astype(np.float64) if flags & B.ALST_FLAG_DW_ACCUMULATE else 0.0
    err = np.abs(r.dW - (base + ref)).max() / top
    # (bf16 +=: the result, up to 5 times max |dW|, is rounded once more: 5 * 2^-9)
    bar = 5e-3 if flags & B.ALST_FLAG_DW_FP32 else 2e-2
    assert r.status == B.ALST_OK and err <= bar, (name, err)
