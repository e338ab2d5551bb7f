"""The ranges dHidden's contraction over the vocabulary is cut into, and the two places of their partial
products (behind the chunk's per-row arrays; the stash rows that the dW group has not reached), against
the oracle with the bars of the parity tests."""
import pytest

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import IGN, _check, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,N,H,V,tile,flags", [
    ("eight_ranges_of_8_k_steps", 300, 128, 4096, 128, 0),
    ("last_range_shorter", 300, 128, 4200, 128, 0),
    ("fewer_k_steps_than_a_range", 300, 128, 500, 128, 0),
    ("two_ranges", 129, 72, 1030, 64, 0),
    # one tile of scratch: no stash rows are left, the other place holds what fits it
    ("one_tile_scratch", 256, 128, 9000, 256, B.ALST_FLAG_TILE_SCRATCH),
    # the last chunk of a group that is full: 2048 rows and one more group of 52
    ("full_group_and_a_short_one", 2100, 64, 3000, 128, 0),
])
def test_ranges(name, N, H, V, tile, flags):
    wl = synth.custom(name, N, H, V, tile, ignore_frac=0.1, seed=71)
    h, W, y = synth.make_inputs(wl)
    f, dH, dW = _oracle(h, W, y)
    r = G.run_fused(h, W, y, tile, flags=flags)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    again = G.run_fused(h, W, y, tile, flags=flags)
    assert (again.dH == r.dH).all()
