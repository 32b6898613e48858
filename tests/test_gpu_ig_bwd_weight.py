"""The weight gradient as one contraction of masked pooled gradients with shifted pixels (rotconv_ig_bwd_weight.hip): tap rows of one
to three groups, both strides, rows around the eight outputs of a lane and the 32 of a step, filters and channels around 16, idx
values that route nothing, and the values the parts do not hold, against the oracle.

Error bar: six part products of 32 outputs a step (the main one cut by at most 2^-23), a few additions in fp32, then sums in 64 bits and
one rounding: a few 2^-24 in norm; 5e-7 is eight.
"""
import numpy as np
import pytest

import parity_util as pu
from oracle import rotconv_oracle as orc
from paper_2512_08888_amd import synth
from test_gpu_ig_bwd_data import _inputs, _rel

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _reference(cfg, x, g, idx):
    dy = orc.orient_maxpool_bwd(np.where(idx < 4, g, 0.0), np.where(idx < 4, idx, 0).astype(np.uint8), cfg.R, cfg.G)
    return orc.reduce_bank_grad(orc.rotconv_bwd_weight(x, dy, cfg.k, cfg.stride, cfg.pad), None, cfg.mode)


CASES = [L(f"v{k}_{stride}_{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, R=4, k=k, stride=stride, pad=pad,
           seed=2500 + i, x_dist="normal")
         for i, (N, Cin, H, W, Cout, k, stride, pad) in enumerate([
             (2, 33, 19, 33, 17, 2, 1, 1), (1, 16, 40, 41, 31, 2, 2, 0), (3, 64, 17, 18, 33, 3, 2, 1), (1, 12, 31, 64, 16, 3, 1, 0),
             (9, 40, 1, 9, 40, 5, 1, 2), (2, 15, 16, 45, 65, 4, 1, 2), (2, 32, 50, 96, 32, 5, 1, 2), (1, 24, 16, 8, 96, 5, 1, 2),
             (1, 97, 17, 29, 31, 5, 2, 2), (1, 10, 30, 20, 12, 6, 1, 3), (2, 8, 64, 64, 32, 7, 1, 3), (1, 70, 16, 28, 16, 7, 2, 3),
             (1, 20, 20, 23, 8, 8, 2, 4), (1, 16, 24, 20, 8, 11, 1, 5), (1, 16, 24, 20, 8, 15, 1, 7), (1, 32, 9, 300, 16, 5, 1, 4)])]


@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_weight_gradient(cfg):
    x, w, g, idx = _inputs(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    assert lay.plan.kernel_name(2) == "mfma_gemm_scatter"
    dw = lay.pool_bwd_weight(g, idx)
    ref = _reference(cfg, x, g, idx)
    assert _rel(dw, ref) < 5e-7
    assert np.array_equal(dw, lay.pool_bwd_weight(g, idx))
    routed = pu.GpuLayer(cfg, x, w, options=dict(gs=1)).pool_bwd_weight(g, idx)          # the gradients through memory
    assert _rel(routed, ref) < 2e-6 and not np.array_equal(dw, routed)


@pytest.mark.parametrize("cfg", [CASES[0], CASES[7], CASES[11]], ids=lambda c: c.name)
def test_weight_gradient_dyadic(cfg):
    x, w, g, idx = _inputs(cfg, dyadic=True)
    assert np.array_equal(pu.GpuLayer(cfg, x, w).pool_bwd_weight(g, idx).astype(np.float64), _reference(cfg, x, g, idx))


@pytest.mark.parametrize("k,stride", [(5, 1), (3, 2)])
def test_values_beyond_the_parts(k, stride):
    """One infinite or NaN gradient: its filter only; products below 2^-100."""
    cfg = L("beyond", N=2, Cin=20, H=21, W=40, Cout=40, R=4, k=k, stride=stride, pad=k // 2, seed=2580, x_dist="normal")
    x, w, g, idx = _inputs(cfg)
    x = np.abs(x) + np.float32(0.5)

    def both(x, g, idx):
        return [pu.GpuLayer(cfg, x, w, options=o).pool_bwd_weight(g, idx) for o in (dict(), dict(gs=-1))]
    for value in (np.inf, -np.inf, np.nan):
        gi, ii = g.copy(), idx.copy()
        gi[0, 33, 5, 11], ii[0, 33, 5, 11] = value, 2
        got, ref = both(x, gi, ii)
        assert np.isfinite(np.delete(got, 33, 1)).all() and not np.isfinite(got[:, 33]).any()
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        ii[0, 33, 5, 11] = 255          # routed nowhere
        got, ref = both(x, gi, ii)
        assert np.isfinite(got).all() and _rel(got, ref) < 1e-5
    got, ref = both(x * np.float32(1e-22), g * np.float32(1e-14), idx)
    assert _rel(got, ref) < 1e-5
