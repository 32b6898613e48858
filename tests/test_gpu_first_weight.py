"""The weight gradient of first layers on bf16 parts (masked pooled gradients times shifted images, turns added afterwards):
row widths around the quads of pixels and the eight quads of a step, one to four channels, filters around a tile (16) and a
wave's two, idx values that route nothing, and the values the parts do not hold, against the oracle.

Error bar: six part products a step (each cut by 2^-23 at the most), a few tens of fp32 additions of partial sums that grow
with the root of their number: sqrt(6 + 40) * 2^-24 in norm is 4e-7; 1e-6 leaves room for the worst of the cases.
"""
import numpy as np
import pytest

import parity_util as pu
from oracle import rotconv_oracle as orc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def _reference(cfg, x, g, idx):
    masked = np.where(idx < 4, g, 0.0)
    dy = orc.orient_maxpool_bwd(masked, np.where(idx < 4, idx, 0).astype(np.uint8), cfg.R, cfg.G)
    return orc.reduce_bank_grad(orc.rotconv_bwd_weight(x, dy, cfg.k, cfg.stride, cfg.pad), None, cfg.mode)


def _inputs(cfg):
    r = np.random.default_rng(cfg.seed)
    idx = r.integers(0, 5, (cfg.N, cfg.Cout, cfg.H, cfg.W)).astype(np.uint8)
    nothing = np.array([4, 7, 8, 12, 15, 127, 128, 254, 255], np.uint8)
    idx = np.where(idx == 4, nothing[r.integers(0, len(nothing), idx.shape)], idx)
    return synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg), idx


CASES = [L(f"w{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, seed=2200 + i, x_dist="normal")
         for i, (N, Cin, H, W, Cout) in enumerate([
             (1, 1, 1, 4, 1), (9, 3, 1, 4, 2), (1, 3, 1, 5, 3), (2, 4, 2, 6, 15), (3, 2, 3, 7, 16), (2, 3, 5, 31, 17),
             (1, 1, 7, 32, 33), (3, 3, 4, 33, 64), (1, 4, 9, 130, 65), (2, 3, 64, 64, 8), (2, 2, 61, 257, 31),
             (4, 3, 256, 256, 40)])]


@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_weight_gradient(cfg):
    x, w, g, idx = _inputs(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    assert lay.plan.kernel_name(2) == "valu_direct"
    dw = lay.pool_bwd_weight(g, idx)
    ref = _reference(cfg, x, g, idx)
    assert _rel(dw, ref) < 1e-6
    assert np.array_equal(dw, lay.pool_bwd_weight(g, idx))
    other = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=-1)).pool_bwd_weight(g, idx)      # the vector-ALU kernel
    assert _rel(other, ref) < 1e-6 and (cfg.N * cfg.H * cfg.W < 100 or not np.array_equal(dw, other))


@pytest.mark.parametrize("scale", [1e-24, 1e24])
def test_magnitudes(scale):
    """Gradients whose products with the pixels leave the parts' range: 1e-48 is no float, 1e-31 is below 2^-100."""
    cfg = L("mag", N=1, Cin=3, H=6, W=73, Cout=6, seed=2250, x_dist="normal")
    x, w, g, idx = _inputs(cfg)
    g = (g * scale).astype(np.float32)
    x = (x * (1e-7 if scale < 1 else 1e10)).astype(np.float32)
    assert _rel(pu.GpuLayer(cfg, x, w).pool_bwd_weight(g, idx), _reference(cfg, x, g, idx)) < 1e-6


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_values_the_parts_do_not_hold(value):
    """One infinite or NaN gradient: its filter only, and signs of infinities as fp32 sums have them."""
    cfg = L("odd", N=2, Cin=3, H=6, W=72, Cout=20, seed=2260, x_dist="normal")
    x, w, g, idx = _inputs(cfg)
    x = np.abs(x) + 0.5
    g[1, 18, 3, 40], idx[1, 18, 3, 40] = value, 1
    dw = pu.GpuLayer(cfg, x, w).pool_bwd_weight(g, idx)
    direct = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=-1)).pool_bwd_weight(g, idx)
    assert np.isfinite(np.delete(dw, 18, 1)).all()
    assert np.array_equal(np.isnan(dw), np.isnan(direct)) and np.array_equal(np.isposinf(dw), np.isposinf(direct))
    idx[1, 18, 3, 40] = 255          # routed nowhere
    assert np.isfinite(pu.GpuLayer(cfg, x, w).pool_bwd_weight(g, idx)).all()
