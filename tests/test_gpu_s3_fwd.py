"""The forward on bf16 parts whose waves own 32 columns of a line of bands (30 of them outputs): row widths around those
counts, odd rows, bands and images that meet inside a wave, the channel and filter remainders, folded banks, incomplete
orientation sets, channel splits, and weights that are not finite, against the oracle.

Error bar: a 32-term instruction cuts six sums per 32 channels, so a sum over K channels and nine taps is within about
sqrt(6 K / 32) * 2^-24 of its value in norm; 1e-6 is four times that for the deepest case (K = 200).
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


def _case(name, N, Cin, H, W, Cout, seed, **k):
    return L(name, N=N, Cin=Cin, H=H, W=W, Cout=Cout, seed=seed, x_dist="normal", **{"R": 4, **k})


CASES = [_case(f"w{w}", 2, 9, 7, w, 18, 1000 + w) for w in (1, 2, 3, 14, 15, 27, 28, 29, 30, 31, 33, 59, 60, 61, 62, 90)] + [
    _case("one_row", 3, 6, 1, 13, 5, 1101),                       # one image row, every band's neighbours outside
    _case("tall", 1, 8, 70, 3, 16, 1102),                         # many bands on a short line
    _case("c31", 1, 31, 6, 21, 16, 1103),
    _case("c33", 1, 33, 6, 21, 17, 1104),                         # a chunk with one channel, a block with one filter
    _case("c96", 2, 96, 9, 40, 16, 1105),                         # three resident chunks
    _case("c160", 1, 160, 5, 75, 3, 1106),
    _case("c161", 1, 161, 5, 75, 20, 1107),                       # streamed
    _case("c200", 3, 200, 4, 26, 16, 1108),                       # streamed, workgroups with waves beyond the line
    _case("wide", 1, 12, 5, 333, 16, 1109),                       # rows of more than 256 pixels
    _case("r1", 1, 24, 6, 19, 7, 1110, R=1),
    _case("r3", 1, 24, 6, 22, 7, 1111, R=3, mode="bilinear"),     # three angles, no whole quarter-turn set
    _case("g4", 2, 24, 9, 23, 10, 1112, R=8, mode="steerable", pool_group=4),
    _case("g2", 1, 16, 6, 25, 6, 1113, pool_group=2),             # groups that cut through the bank
    _case("fold2", 1, 36, 6, 22, 11, 1114, R=8, mode="steerable"),
    _case("fold4", 2, 36, 6, 22, 7, 1115, R=16, mode="bilinear"),
    _case("fold4s", 1, 170, 3, 18, 6, 1116, R=16, mode="bilinear"),
]


@pytest.mark.parametrize("cfg,csplit", [pytest.param(c, s, id=f"{c.name}-{s}") for c in CASES for s in (0, 1, 3) if s < 3 or c.Cin > 64])
def test_forward(cfg, csplit):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=csplit, fwd_base=-1))
    assert lay.plan.kernel_name(0) == "mfma_p4" and lay.plan.bf16_parts(0)
    yp, idx = lay.pool_fwd()
    assert _rel(yp, ref["ypool"]) < 1e-6
    pu.check_idx(idx, ref["y"], ref["abs_terms"], cfg.G, cfg.name)
    yu = lay.nan(lay.U)
    rc.rotconv_fwd(lay.plan, lay.x, lay.w, yu)
    assert _rel(yu.cpu().numpy(), ref["y"].reshape(yu.shape)) < 1e-6


@pytest.mark.parametrize("W", [16, 29, 62])
@pytest.mark.parametrize("tap", [0, 1, 5, 8])
def test_weights_that_are_not_finite_do_not_reach_through_the_padding(W, tap):
    """One orientation: an infinite weight makes exactly those outputs NaN whose window holds a pixel at its tap."""
    cfg = _case("inf", 2, 8, 9, W, 4, 1200, R=1)
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    w[0, 1, 3, tap // 3, tap % 3] = np.inf
    lay = pu.GpuLayer(cfg, x, w)
    yu = lay.nan(lay.U)
    rc.rotconv_fwd(lay.plan, lay.x, lay.w, yu)
    bad = ~np.isfinite(yu.cpu().numpy())
    want = np.zeros(bad.shape, bool)
    dy, dx = tap // 3 - 1, tap % 3 - 1
    want[:, 1, max(0, -dy):9 - max(0, dy), max(0, -dx):W - max(0, dx)] = True
    assert np.array_equal(bad, want)


UNALIGNED = [
    (_case("wide", 2, 9, 5, 300, 7, 1301), {}),                    # a row of more than 256 pixels, no whole waves
    (_case("narrow", 1, 40, 7, 18, 5, 1302), {}),
    (_case("odd", 1, 40, 7, 21, 5, 1303), {}),
    (_case("split", 1, 96, 6, 18, 5, 1304), dict(fwd_csplit=3)),
    (_case("fold", 1, 36, 6, 22, 11, 1305, R=8, mode="steerable"), dict(fwd_base=-1)),
    (_case("partial", 1, 24, 6, 300, 7, 1306, R=6, mode="bilinear"), dict(fwd_base=-1)),
    (_case("cut", 1, 16, 6, 26, 6, 1307, pool_group=2), {}),
    (_case("chain_split", 2, 96, 6, 64, 5, 1308), dict(fwd_csplit=3)),     # waves chained over the row: x at eight bytes
]


@pytest.mark.parametrize("cfg,opt", UNALIGNED, ids=[c.name for c, _ in UNALIGNED])
def test_tensors_off_their_alignment_take_the_same_kernel(cfg, opt):
    """An image out of a batch: bit for bit the result on aligned tensors (the generic kernels add up in another order)."""
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w, options=opt)
    step = 2 if cfg.name == "chain_split" else 1

    def run(off):
        def at(shape, dt, v):
            n = int(np.prod(shape))
            return torch.full((n + off,), v, dtype=dt, device="cuda")[off:].view(shape)
        xd, yp, idx, yu = at(x.shape, torch.float32, 0.), at(lay.P, torch.float32, np.nan), at(lay.P, torch.uint8, 254), at(lay.U, torch.float32, np.nan)
        xd.copy_(lay.x)
        rc.rotconv_pool_fwd(lay.plan, xd, lay.w, yp, idx)
        rc.rotconv_fwd(lay.plan, xd, lay.w, yu)
        return yp, idx, yu

    want = run(0)
    ref = pu.oracle_layer(cfg, x, w, g)
    assert _rel(want[0].cpu().numpy(), ref["ypool"]) < 1e-6
    for off in (step, 3 * step):
        got = run(off)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2], want[2]), off
