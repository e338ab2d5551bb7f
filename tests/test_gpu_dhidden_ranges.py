"""The ranges dHidden's contraction over the vocabulary is cut into, and the two places of their partial
products (behind the chunk's per-row arrays; the stash rows that the dW group has not reached), against
the oracle with the bars of the parity tests.  `ranges` and `stash` are what each chunk of the call is to
have, as the library's own host functions give it."""
import pytest

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import IGN, _check, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,N,H,V,tile,flags,frac,ranges,stash", [
    ("eight_ranges_of_8_k_steps", 300, 128, 4096, 128, 0, 0.1, [8], [1]),
    ("last_range_shorter", 300, 128, 4200, 128, 0, 0.1, [8], [1]),
    ("fewer_k_steps_than_a_range", 300, 128, 500, 128, 0, 0.1, [1], [1]),
    ("two_ranges", 129, 72, 1030, 64, 0, 0.1, [2], [1]),
    # one tile of scratch: no stash rows are left, the other place holds what fits it
    ("one_tile_scratch", 256, 128, 9000, 256, B.ALST_FLAG_TILE_SCRATCH, 0.1, [3], [0]),
    # a group of 2048 rows in three chunks, the last of which finds no room for partial products, and one
    # more group of 52
    ("full_group_and_a_short_one", 2100, 64, 3000, 128, 0, 0.0, [6, 6, 1, 6], [1, 1, 0, 1]),
    # dense rows end inside the first group: the second has none
    ("dense_rows_end_before_the_last_group", 2100, 64, 3000, 128, 0, 0.1, [6, 6, 1, 1], [1, 1, 0, 1]),
])
def test_ranges(name, N, H, V, tile, flags, frac, ranges, stash):
    wl = synth.custom(name, N, H, V, tile, ignore_frac=frac, seed=71)
    h, W, y = synth.make_inputs(wl)
    chunks = G.ce_chunks(N, H, V, tile, flags, int((y != IGN).sum()))
    assert [c.ranges for c in chunks] == ranges and [c.in_stash for c in chunks] == stash
    assert all(c.added_up for c in chunks if c.ranges > 1)
    f, dH, dW = _oracle(h, W, y)
    r = G.run_fused(h, W, y, tile, flags=flags)
    _check(r, f, dH, dW, name, valid=(y != IGN))
    again = G.run_fused(h, W, y, tile, flags=flags)
    assert (again.dH == r.dH).all()
