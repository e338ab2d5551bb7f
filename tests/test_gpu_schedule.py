"""The launch schedule of the cross-entropy path: chunks of dense rows that span several of the
caller's tiles, dW groups, and the two ways the rows are numbered, against the oracle."""
import numpy as np
import pytest

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import IGN, _check, _oracle

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, H, V, tile, ignore_frac, flags
    # few columns of H per vocabulary id: the scratch of one tile holds the partials of two tiles'
    # rows, so a dW group of 8 tiles is several chunks, the last of them shorter
    ("several_chunks_per_group", 1700, 64, 16640, 128, 0.1, 0),
    ("several_groups_last_one_short", 2300, 64, 520, 128, 0.1, 0),
    ("one_tile_scratch_tiles_of_100", 700, 72, 520, 100, 0.2, B.ALST_FLAG_TILE_SCRATCH),
    # dense rows end in an earlier chunk than the sequence: the last chunk has none
    ("last_chunk_empty", 2300, 64, 520, 256, 0.6, 0),
    # more rows than the one-workgroup numbering takes; exactly as many as it takes
    ("numbered_by_many_workgroups", 33000, 8, 40, 8192, 0.1, 0),
    ("numbered_by_one_workgroup", 32768, 8, 40, 8192, 0.1, 0),
]


@pytest.mark.parametrize("name,N,H,V,tile,frac,flags", CASES, ids=[c[0] for c in CASES])
def test_chunks_and_groups_match_oracle(name, N, H, V, tile, frac, flags):
    wl = synth.custom(name, N, H, V, tile, ignore_frac=frac, seed=61)
    h, W, y = synth.make_inputs(wl)
    f, dH, dW = _oracle(h, W, y)
    r = G.run_fused(h, W, y, tile, flags=flags)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    assert (r.dH[y == IGN] == 0.0).all()
    s = G.run_split(h, W, y, tile, flags=flags)
    assert s.status_bwd == B.ALST_OK and s.loss_bits == r.loss_bits
    _check(s, f, dH, dW, name + " split", valid=(y != IGN))
    assert (s.lse.view(np.uint32) == r.lse.view(np.uint32)).all()
