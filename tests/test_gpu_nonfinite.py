"""Infinities and NaN in the kernels of short calls (small blocks): what is in a row of an ignored token reaches nothing, what is in a
row that takes part reaches that row's outputs only (a block reads the last row in place of those it lacks).  Sigmoids at both ends.
Against the fp64 oracle, bar as in the other parity tests: 2e-2 of max |ref| per output; lse 1e-3."""
import numpy as np
import pytest
import torch

from oracle import tiled_ce_oracle as orc
from oracle import tiled_mlp_oracle as morc
from paper_2506_13996_amd import binding as B
from paper_2506_13996_amd import synth
from tests import gpu_util as G
from tests import test_gpu_mlp as TM
from tests.test_gpu_parity import IGN

pytestmark = pytest.mark.gpu
TOL = 2e-2
INF, NINF, NAN = 0x7f80, 0xff80, 0x7fc0                # bf16


@pytest.mark.parametrize("N,H,V", [(300, 72, 500), (1000, 256, 1000)])
@pytest.mark.parametrize("bits", [INF, NINF, NAN])
def test_cross_entropy(N, H, V, bits):
    wl = synth.custom("nonfinite", N, H, V, 1024, ignore_frac=0.2, seed=91)
    h, W, y = synth.make_inputs(wl)
    y[N // 3], y[-1] = IGN, 5
    i = B.alst_debug_ce_chunk(N, H, V, 1024, 0, 0, int((y != IGN).sum()))
    assert i.logits_columns and i.dhidden_columns and i.dw_columns and i.numbered_by_gather
    f, (dH, dW) = orc.forward(h, W, y), orc.backward(h, W, y)
    bad = h.copy()
    bad[y == IGN] = bits                               # ignored rows: whole rows of it
    r = G.run_fused(bad, W, y, 1024)
    assert r.status == B.ALST_OK and abs(r.loss - f["loss"]) <= 1e-3 * abs(f["loss"])
    assert G.grad_err(r.dH, dH) <= TOL and G.grad_err(r.dW, dW) <= TOL
    bad[-1, 3] = bits                                  # the last row, which takes part
    r = G.run_fused(bad, W, y, 1024)
    assert r.status == B.ALST_ERR_NONFINITE and not np.isfinite(r.loss)
    others = (y != IGN) & (np.arange(N) < N - 1)
    assert np.abs(r.lse[others] - f["lse"][others]).max() <= 1e-3 * np.abs(f["lse"][others]).max()
    assert G.grad_err(r.dH[:-1], dH[:-1]) <= TOL
    assert not np.isfinite(r.dH[-1]).all() and not np.isfinite(r.dW).all()


@pytest.mark.parametrize("N,H,I", [(300, 72, 200), (500, 320, 448), (300, 64, 1720)])
@pytest.mark.parametrize("bits", [INF, NINF, NAN])
def test_mlp(N, H, I, bits):
    assert B.alst_debug_layer(1, N, H, I, 2048).gated_columns
    wl = synth.MlpWorkload("nonfinite", N, H, I, 2048, seed=92)
    x, Wg, Wu, Wd, dy = synth.make_mlp_inputs(wl)
    ref_y, ref_dx = morc.forward(x, Wg, Wu, Wd, row_block=256), morc.backward(x, Wg, Wu, Wd, dy, row_block=256)[0]
    for at in (x, dy):
        good = at.copy()
        at[-1, 3] = bits
        y, dx, gW = TM._run(x, Wg, Wu, Wd, dy, 2048)
        assert G.grad_err(y[:-1], ref_y[:-1]) <= TOL and G.grad_err(dx[:-1], ref_dx[:-1]) <= TOL
        assert not np.isfinite(dx[-1]).all() and not any(np.isfinite(g).all() for g in gW[:2])
        if at is x:
            assert not np.isfinite(y[-1]).all()
        else:
            assert G.grad_err(y, ref_y) <= TOL
        at[:] = good


@pytest.mark.parametrize("N,H,I", [(192, 64, 128), (1032, 72, 1032)])
def test_sigmoid_at_both_ends(N, H, I):
    """Gates far out: silu is 0 or the gate, its derivative 0 or 1, nothing is NaN."""
    gates = np.array([-3e38, -1e30, -200.0, -89.0, 0.0, 20.0, 200.0, 2.0 ** 100])
    bits = lambda t: synth.f32_to_bf16_bits(t.astype(np.float32))
    x, Wg, Wu = np.zeros((N, H)), np.zeros((I, H)), np.zeros((I, H))
    Wd, dy = np.zeros((H, I)), np.zeros((N, H))
    g = orc.bf16_bits_to_f64(bits(gates))[np.arange(N) % len(gates)]
    x[:, 0], x[:, 1], Wg[:, 0], Wu[:, 1] = g, 1.0, 1.0, 0.5
    Wd[3], dy[:, 3] = 2.0 ** -10, 1.0
    y, dx, _ = TM._run(bits(x), bits(Wg), bits(Wu), bits(Wd), bits(dy), 2048)
    with np.errstate(over="ignore"):
        sg = 1.0 / (1.0 + np.exp(-g))
    silu, da = g * sg, 2.0 ** -10
    for got, ref in ((y[:, 3], I * 2.0 ** -10 * silu * 0.5), (dx[:, 0], I * da * 0.5 * sg * (1.0 + g * (1.0 - sg))),
                     (dx[:, 1], I * da * silu * 0.5)):
        assert np.isfinite(got).all()
        assert (np.abs(got - ref) <= TOL * np.abs(ref) + 1e-30).all()
