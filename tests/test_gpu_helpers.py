"""The small kernels around the large ones at their edges: the sum of split weight gradients that is turned round on its way
to dw (channels that are no multiple of its 64, one and two base banks, the routed-gradient table), and the 1x1 head whose
channels are shared out over waves and workgroups (fewer channels than waves, the most it takes, a pixel vector or two).

Bars: fp32 sums of n products are within about sqrt(n) 2^-24 of their norm (n at most 4096: 4e-6), bf16 outputs one
rounding, 2^-9.
"""
import numpy as np
import pytest
import torch

import parity_util as pu
from oracle import unet_oracle as uo
from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


WIDE = [
    L("d_200", N=2, Cin=200, H=12, W=16, Cout=160, R=4, x_dist="normal", seed=1301),
    L("d_321", N=2, Cin=321, H=8, W=16, Cout=96, R=1, x_dist="normal", seed=1302),
    L("d_steer", N=2, Cin=192, H=8, W=16, Cout=160, R=8, mode="steerable", pool_group=4, x_dist="normal", seed=1303),
    L("d_table", N=2, Cin=260, H=8, W=16, Cout=144, R=16, mode="bilinear", x_dist="normal", seed=1304),
]


@pytest.mark.parametrize("cfg", WIDE, ids=[c.name for c in WIDE])
def test_wide_weight_gradient(cfg):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    ref = pu.oracle_layer(cfg, x, w, g)
    dw = lay.pool_bwd_weight(g, ref["idx"].astype(np.uint8))
    assert _rel(dw, ref["dw"]) < 4e-6


@pytest.mark.parametrize("bf", [False, True])
@pytest.mark.parametrize("N,Cin,Cout,P", [(1, 1, 1, 8), (2, 3, 8, 16), (1, 5, 2, 264), (3, 65, 7, 520), (1, 1024, 8, 72), (2, 64, 6, 8200)])
def test_head(N, Cin, Cout, P, bf):
    rng = np.random.default_rng(Cin)
    dt = torch.bfloat16 if bf else torch.float32
    t = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(dt)
    x, w, dy = t(N, Cin, 1, P), t(Cout, Cin), t(N, Cout, 1, P)
    f = lambda v: v.float().numpy()
    bar = 5e-3 if bf else 4e-6
    y, dx = torch.full((N, Cout, 1, P), float("nan"), dtype=dt, device="cuda"), torch.full((N, Cin, 1, P), float("nan"), dtype=dt, device="cuda")
    dw = torch.full((Cout, Cin), float("nan"), device="cuda")
    ws = torch.empty(max(256, rc.glue_conv1x1_workspace_bytes(N, Cin, Cout, P)), dtype=torch.uint8, device="cuda")
    rc.glue_conv1x1_fwd(x.cuda(), w.cuda(), y)
    rc.glue_conv1x1_bwd_data(dy.cuda(), w.cuda(), dx)
    rc.glue_conv1x1_bwd_weight(x.cuda(), dy.cuda(), dw, ws)
    assert _rel(y.float().cpu().numpy(), uo.conv1x1_fwd(f(x), f(w))) < bar
    dxr, dwr = uo.conv1x1_bwd(f(x), f(w), f(dy))
    assert _rel(dx.float().cpu().numpy(), dxr) < bar
    assert _rel(dw.cpu().numpy(), dwr) < 4e-6
