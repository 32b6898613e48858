"""The pooled forward on products of the base bank as bf16 parts (rotconv_p4_fwd_base_kernel.h): chunks of 32 channels, blocks of 16
filters, resident (one to three banks' sums parked) and streamed, whole rows and rows with masks, every chain length, and the values
the parts do not hold, against the oracle and the fp32 instructions (plan option bf16_parts = -1).

Error bar: a chunk's products are one cut sum, the chunks', the bank's (up to four base products) and the nine taps' sums are
roundings in fp32: sqrt(chunks + 3 + 9 / 2) * 2^-24 in norm; four times that.
"""
import numpy as np
import pytest

import parity_util as pu
from oracle import rotconv_oracle as orc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig

LAYERS = [L(f"b{R}_{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, R=R, mode="p4m" if p4m else "bilinear",
            x_dist="normal", seed=2600 + i)
          for i, (N, Cin, H, W, Cout, R, p4m) in enumerate([
              (1, 5, 9, 16, 16, 16, False), (2, 32, 7, 30, 17, 16, False), (1, 64, 12, 64, 33, 16, False), (1, 65, 26, 40, 16, 16, False),
              (2, 96, 9, 128, 16, 16, False), (1, 128, 31, 34, 20, 16, False), (1, 129, 32, 32, 16, 16, False), (1, 161, 57, 18, 16, 16, False),
              (1, 256, 40, 32, 32, 16, False), (2, 24, 19, 8, 40, 8, False), (1, 160, 9, 128, 17, 8, False), (1, 161, 33, 50, 16, 8, False),
              (1, 40, 8, 144, 16, 8, False), (2, 33, 9, 24, 18, 8, True), (1, 200, 32, 64, 16, 8, True)])]


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("cfg", LAYERS, ids=[c.name for c in LAYERS])
def test_against_the_oracle(cfg, relu):
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y, yp, _, w_rot = orc.layer_fwd(x, w, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    lay = pu.GpuLayer(cfg, x, w, relu=relu)
    assert lay.plan.kernel_name(0) == "mfma_p4_base"
    got, idx = lay.pool_fwd()
    bar = 4 * 2.0 ** -24 * np.sqrt((cfg.Cin + 31) // 32 + 7.5)
    if relu:
        dead, sure = yp <= 0, np.abs(yp) > 1e-5 * np.abs(yp).max()
        assert np.array_equal((idx == 255)[sure], dead[sure]) and _rel(got, np.where(dead, 0, yp)) < bar
        return
    assert _rel(got, yp) < bar
    pu.check_idx(idx, y, orc.rotconv_fwd(np.abs(x), np.abs(w_rot), cfg.stride, cfg.pad), cfg.G, cfg.name)


@pytest.mark.parametrize("cfg", [LAYERS[1], LAYERS[8], LAYERS[13]], ids=lambda c: c.name)
def test_values_the_parts_do_not_hold(cfg):
    """Infinite, huge and tiny pixels and an infinite weight come out as on the fp32 instructions: non-finite where those
    are, within 1e-6 elsewhere (both forms are within the bar above of the same sum)."""
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y, px = cfg.H // 2, cfg.W // 2

    def both(x, w):
        return [pu.GpuLayer(cfg, x, w, options=o).pool_fwd()[0] for o in (None, dict(bf16_parts=-1))]

    for bad in (np.inf, -np.inf, 3.4e38, 1e38, -2.0 ** 120):
        xb = x.copy()
        xb[0, 2, y, px] = bad
        got, ref = both(xb, w)
        fin = np.isfinite(ref)
        assert np.array_equal(got[~fin], ref[~fin], equal_nan=True) and np.isfinite(got[fin]).all()
        assert _rel(got[fin].astype(np.float64) / 2.0 ** 100, ref[fin].astype(np.float64) / 2.0 ** 100) < 1e-6
    wb = w.copy()
    wb.reshape(-1)[4] = np.inf
    got, ref = both(x, wb)
    fin = np.isfinite(ref)
    assert np.array_equal(got[~fin], ref[~fin], equal_nan=True) and _rel(got[fin], ref[fin]) < 1e-6
    for ex, ew in ((-75, -40), (-115, 0), (60, 40)):
        got, ref = both(np.ldexp(x, ex), np.ldexp(w, ew))
        assert _rel(np.ldexp(got.astype(np.float64), -ex - ew), np.ldexp(ref.astype(np.float64), -ex - ew)) < 1e-6


@pytest.mark.parametrize("cfg", [LAYERS[1], LAYERS[4], LAYERS[8], LAYERS[13]], ids=lambda c: c.name)
def test_small_values_beside_ordinary_ones(cfg):
    """Pixels that the parts hold to a few bits only (2^-122 of a part that ends at 2^-134), three by three among ordinary ones at every
    offset from a lane's four pixels: what draws on them alone is as on the fp32 instructions.  Both are within the bar at the
    top of the same sum (128 channels, 7e-7)."""
    x, w = synth.make_x(cfg), np.ldexp(synth.make_w(cfg), 8)
    at = [(2, 4 * i + i % 4) for i in range(1, (cfg.W - 3) // 4)]
    for y, c in at:
        x[..., y:y + 3, c:c + 3] = np.ldexp(x[..., y:y + 3, c:c + 3], -122)
    got, ref = (np.stack([pu.GpuLayer(cfg, x, w, options=o).pool_fwd()[0][..., y + 1, c + 1] for y, c in at])
                for o in (None, dict(bf16_parts=-1)))
    assert 0 < np.abs(ref).max() < 2.0 ** -100
    assert _rel(np.ldexp(got.astype(np.float64), 120), np.ldexp(ref.astype(np.float64), 120)) < 1e-6
