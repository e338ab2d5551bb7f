"""The fp64 sum behind the loss is formed in one order, whichever launch makes it (a kernel of its own, or a workgroup of
the launch that adds up the last chunk's ranges of dHidden): its bits, which tell two orders apart where those of the fp32 loss
seldom do, are the same for every tile and entry point and those of a fixed sum on the host.

Of terms of one size every order is exact in fp64.  Here one term is 80 and the others, 2^-48 to 2^-49 (1 to 2), are each less than half a
last place of it: added to it one by one they are lost, added up first they are not.  A row's logits are t for word 0 and -80 for all others;
with t that small the sum of exponentials is 1, the term of a row with label 0 is -t and that of another label 80, exactly."""
import numpy as np
import pytest
import torch

from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests.test_gpu_parity import IGN

pytestmark = pytest.mark.gpu


def _host_sum(terms, lanes=1024):
    """1024 sums of every 1024th term, added up pairwise."""
    rows = -(-len(terms) // lanes)
    part = np.zeros(lanes)
    for row in np.pad(terms.astype(np.float64), (0, rows * lanes - len(terms))).reshape(rows, lanes):
        part += row
    w = lanes // 2
    while w:
        part[:w] += part[w:2 * w]
        w //= 2
    return part[0]


@pytest.mark.parametrize("N,H,V", [(2048, 256, 1000), (1, 64, 300), (700, 64, 1000), (5121, 64, 2000), (16384, 8, 1024), (16385, 8, 1024)])
def test_loss_sum_is_formed_in_one_order(N, H, V):
    rng = np.random.default_rng(81)
    h, W = np.zeros((N, H), np.float32), np.zeros((V, H), np.float32)
    h[:, 0], h[:, 1] = -rng.uniform(1, 2, N) * np.exp2(-rng.integers(48, 50, N)), 1.0
    W[0, 0], W[1:, 1] = 1.0, -80.0
    y = np.where(rng.random(N) < 0.1, IGN, 0).astype(np.int32)
    y[0] = 5
    h, W = synth.f32_to_bf16_bits(h), synth.f32_to_bf16_bits(W)
    hd, Wd, yd = G.bits_to_dev(h), G.bits_to_dev(W), torch.from_numpy(y).cuda()
    seen, added_up = set(), set()
    for tile in (128, 256, 512, 2048):
        last = G.ce_chunks(N, H, V, tile, 0, N)[-1]
        added_up.add(last.added_up)
        for fused in (True, False):
            ws = B.alloc_workspace(N, H, V, tile)
            loss, lse = torch.zeros(1, device="cuda"), torch.zeros(N, device="cuda")
            if fused:
                dH, dW = torch.empty_like(hd), torch.empty_like(Wd)
                B.alst_tiled_ce_forward_backward(hd, Wd, yd, tile, IGN, loss_out=loss, lse_out=lse, dHidden=dH, dW=dW,
                                                 workspace=ws)
            else:
                B.alst_tiled_ce_forward(hd, Wd, yd, tile, IGN, loss_out=loss, lse_out=lse, workspace=ws)
            terms = torch.empty(N, device="cuda")
            B.alst_tiled_ce_token_losses(ws, N, H, V, tile, terms)
            torch.cuda.synchronize()
            # the workspace begins with status, padding, the valid count, g / M, padding and the sum
            loss_sum = np.frombuffer(ws[24:32].cpu().numpy().tobytes(), np.float64)[0]
            assert loss_sum == _host_sum(terms.cpu().numpy()), (tile, fused, last.added_up)
            seen.add((loss_sum.tobytes(), loss.cpu().numpy().tobytes()))
    assert len(seen) == 1
    if (N, H, V) == (2048, 256, 1000):
        assert added_up == {0, 1}              # both launches are met
    if N > 1024:                               # (the order matters)
        terms = terms.cpu().numpy()
        assert len({_host_sum(terms, lanes) for lanes in (256, 1024)}) == 2
