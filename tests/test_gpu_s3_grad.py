"""Both gradients on bf16 parts where their rules take layers that used to run on fp32 instructions or on padded rows: rows of
any width (pieces of four pixels that end beyond the row, odd rows, rows narrower than a strip), 17 to 32 channels, and input
gradients of few channels, against the oracle, with a third of the winners dead (byte 255).  Tensors one element off their
alignment go the same way where the kernel loads pixel by pixel.

Error bar: six sums per 16 products, each cut by up to half an ulp, in sums of up to n = 4000 products: sqrt(6 n / 16) 2^-25 =
1.2e-6 of the norm at the most; twice that is asked for.
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


def _case(N, Cin, H, W, Cout, seed, **k):
    return L(f"g{Cin}x{H}x{W}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, seed=seed, x_dist="normal", **{"R": 4, **k})


CASES = [_case(2, 20, 9, w, 18, 1500 + w) for w in (1, 2, 3, 5, 15, 17, 18, 30, 31, 33, 47)] + [
    _case(1, 17, 8, 16, 5, 1601), _case(1, 32, 7, 20, 33, 1602), _case(3, 33, 5, 19, 16, 1603), _case(1, 65, 1, 21, 40, 1604),
    _case(1, 129, 6, 13, 9, 1605), _case(2, 3, 12, 22, 8, 1606, R=8, mode="steerable", pool_group=4),
    _case(2, 24, 10, 27, 10, 1607, R=8, mode="steerable", pool_group=4), _case(1, 40, 9, 25, 12, 1608, R=1)]


@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_gradients(cfg):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    assert lay.plan.bf16_parts(1) == (cfg.W % 2 == 1 or cfg.Cin <= 4) and lay.plan.bf16_parts(2) == (cfg.Cin > 16)
    rng = np.random.default_rng(cfg.seed)
    ng = cfg.R // cfg.G
    idx = (rng.integers(0, cfg.G, lay.P) * ng + np.arange(lay.P[1]).reshape(1, -1, 1, 1) % ng).astype(np.uint8)
    off = rng.random(lay.P) < 1 / 3
    routed = np.where(off, 255, idx).astype(np.uint8)
    dxr, dwr = orc.layer_bwd(x, w, np.where(off, 0, g), idx, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    assert _rel(lay.pool_bwd_data(g, routed), dxr) < 2.4e-6
    assert _rel(lay.pool_bwd_weight(g, routed), dwr) < 2.4e-6


@pytest.mark.parametrize("W", [21, 18])
def test_unaligned_tensors(W):
    cfg = _case(1, 20, 6, W, 8, 1700)
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    idx = np.random.default_rng(1).integers(0, 4, lay.P).astype(np.uint8)

    def off(a, dt=torch.float32):
        t = torch.zeros(a.size + 1, dtype=dt, device="cuda")[1:].view(a.shape)
        t.copy_(torch.from_numpy(a))
        return t

    xd, gd, id_ = off(x), off(g.astype(np.float32)), off(idx, torch.uint8)
    dx, dw = off(np.full(x.shape, np.nan, np.float32)), torch.full(w.shape, float("nan"), device="cuda")
    rc.rotconv_pool_bwd_data(lay.plan, gd, id_, lay.w, dx)
    rc.rotconv_pool_bwd_weight(lay.plan, xd, gd, id_, dw)
    dxr, dwr = orc.layer_bwd(x, w, g, idx, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    assert _rel(dx.cpu().numpy(), dxr) < 2.4e-6 and _rel(dw.cpu().numpy(), dwr) < 2.4e-6
