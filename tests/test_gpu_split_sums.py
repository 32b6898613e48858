"""Split contractions of odd rows, whose parts are summed four floats at a time: an odd number of elements (the parts start at
any float), results one float off their alignment.  Against the oracle, and bit for bit what aligned results hold.

Error bar: n products in norm within about sqrt(6 n / 16) 2^-24: 3e-6 for the 9 * 512 here.
"""
import numpy as np
import pytest
import torch

import parity_util as pu
from oracle import rotconv_oracle as orc
from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def _nan(shape, off):
    return torch.full((int(np.prod(shape)) + off,), float("nan"), device="cuda")[off:].view(shape)


CASES = [
    L("odd_3", N=1, Cin=201, H=7, W=9, Cout=5, R=1, x_dist="normal", seed=2301),               # 315 outputs
    L("odd_1", N=3, Cin=97, H=5, W=13, Cout=3, R=3, mode="bilinear", x_dist="normal", seed=2302),  # 1755
    L("even_2", N=1, Cin=97, H=5, W=6, Cout=3, R=1, x_dist="normal", seed=2303),               # 90: parts at eight bytes
]


@pytest.mark.parametrize("csplit", [2, 3])
@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_forward(cfg, csplit):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=csplit))
    out = []
    for off in (0, 1, 2, 3) if cfg.W % 2 else (0,):
        y = _nan(lay.U, off)
        rc.rotconv_fwd(lay.plan, lay.x, lay.w, y)
        out.append(y.cpu().numpy())
        assert np.array_equal(out[0], out[-1]), off
    assert _rel(out[0], ref["y"].reshape(lay.U)) < 3e-6


@pytest.mark.parametrize("W", [9, 10])
def test_input_gradient(W):
    """512 filters on a map of three strips: shared out over many workgroups (33 x 7 x 9 elements: odd; x 10: twice an odd number)."""
    cfg = L("dx", N=1, Cin=33, H=7, W=W, Cout=512, R=4, x_dist="normal", seed=2304)
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=1))
    idx = np.random.default_rng(1).integers(0, 4, lay.P).astype(np.uint8)
    ref = orc.layer_bwd(x, w, g, idx, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)[0]
    gd, id_, out = pu.dev(g, torch.float32), pu.dev(idx), []
    for off in (0, 1, 2, 3) if W % 2 else (0,):
        dx = _nan(x.shape, off)
        rc.rotconv_pool_bwd_data(lay.plan, gd, id_, lay.w, dx)
        out.append(dx.cpu().numpy())
        assert np.array_equal(out[0], out[-1]), off
    assert _rel(out[0], ref) < 3e-6
