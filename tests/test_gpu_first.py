"""The pooled forward of first layers on bf16 parts (all four turns of a filter as rows of one contraction over channels and
taps): row widths around the sixteen quads of pixels of a wave, one to three channels, filters around a tile (4) and a
workgroup (64), and the values the parts do not hold, against the oracle.

Error bar: one 32-term instruction per part product, six of them: sqrt(6) * 2^-24 in norm; 6e-7 is four times that.
"""
import numpy as np
import pytest
import torch

import parity_util as pu
from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


CASES = [L(f"f{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, seed=2000 + i, x_dist="normal")
         for i, (N, Cin, H, W, Cout) in enumerate([
             (1, 1, 1, 4, 1), (1, 3, 1, 8, 3), (2, 3, 2, 4, 4), (3, 2, 3, 12, 5), (1, 3, 5, 60, 63), (2, 1, 7, 64, 64),
             (1, 3, 4, 68, 65), (1, 2, 9, 132, 7), (2, 3, 33, 20, 130), (2, 3, 300, 256, 9)])]


@pytest.mark.parametrize("relu", [0, 1])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_forward(cfg, relu):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w, relu=bool(relu))
    assert lay.plan.kernel_name(0) == "valu_direct" and lay.plan.bf16_parts(0)
    yp, idx = lay.pool_fwd()
    dead = ref["ypool"] <= 0
    if relu:
        assert _rel(yp, np.where(dead, 0, ref["ypool"])) < 6e-7
        sure = np.abs(ref["ypool"]) > 1e-5 * np.abs(ref["ypool"]).max()
        assert np.array_equal((idx == 255)[sure], dead[sure])
        other = pu.GpuLayer(cfg, x, w, relu=bool(relu), options=dict(direct_ty=1)).pool_fwd()[1]      # the vector-ALU kernel
        assert np.mean(idx == other) > 0.999
    else:
        assert _rel(yp, ref["ypool"]) < 6e-7
        pu.check_idx(idx, ref["y"], ref["abs_terms"], cfg.G, cfg.name)


@pytest.mark.parametrize("where", ["x", "w"])
def test_values_beyond_the_parts(where):
    """1e25 and infinity: summed in fp32, as by the vector-ALU kernel; positions outside the image reach nothing."""
    cfg = L("odd", N=1, Cin=3, H=6, W=72, Cout=6, seed=2100, x_dist="normal")
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    if where == "x":
        x[0, 1, 2, 70] = 1e25
    else:
        w[0, 2, 1, 0, 2] = 1e25
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w)
    yp, _ = lay.pool_fwd()
    big = np.abs(ref["ypool"]) > 1e15
    for part in (big, ~big):
        assert _rel(yp[part], ref["ypool"][part]) < 6e-7
    if where == "x":
        x[0, 1, 2, 70] = np.inf
        yp, _ = pu.GpuLayer(cfg, x, w).pool_fwd()
        window = np.zeros(yp.shape, bool)
        window[:, :, 1:4, 69:72] = True
        assert np.isfinite(yp[~window]).all() and not np.isfinite(yp[window]).any()
        assert np.isposinf(yp[window]).any()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("at", [(0, 0), (2, 5), (5, 71)])
def test_nan(at, relu):
    """A NaN pixel makes NaN what it reaches in the instruction's sums, a NaN weight its filter (which is summed in fp32)."""
    cfg = L("nan", N=1, Cin=3, H=6, W=72, Cout=6, seed=2110, x_dist="normal")
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    x[0, 1, at[0], at[1]] = np.nan
    lay = pu.GpuLayer(cfg, x, w, relu=relu)
    assert lay.plan.bf16_parts(0)
    yp, _ = lay.pool_fwd()
    window = np.zeros(yp.shape, bool)
    window[:, :, max(0, at[0] - 1):at[0] + 2, max(0, at[1] - 1):at[1] + 2] = True
    assert np.isnan(yp[window]).all() and np.isfinite(yp[~window]).all()
    x[0, 1, at[0], at[1]] = 0
    w[0, 4, 1, 1, 1] = np.nan
    yp, _ = pu.GpuLayer(cfg, x, w, relu=relu).pool_fwd()
    assert np.isnan(yp[:, 4]).all() and np.isfinite(np.delete(yp, 4, 1)).all()
