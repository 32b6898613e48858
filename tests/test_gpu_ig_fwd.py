"""The forward as one contraction over channels and taps (rotconv_ig_fwd.hip): filters of other sizes and strides with the four
turns pooled, and single orientations, around tiles (16 filters, 64 to 256 pixels), chunks of 32 channels, orbits of taps with and
without a centre, shares of channels and orbits, and the values the parts do not hold, against the oracle.

Error bar: per tap and chunk one cut sum of 32 products (2^-24 of it), then additions in fp32 over the k^2 taps and over the chunks,
each a rounding of a partial sum that grows with the root of their number: sqrt(1 + (k^2 + chunks) / 2) * 2^-24 in norm; four times that.
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
    ref = np.asarray(ref, np.float64)
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def _bar(cfg):
    return 4 * 2.0 ** -24 * np.sqrt(1 + (cfg.k ** 2 + (cfg.Cin + 31) // 32) / 2)


TURNS = [L(f"t{k}_{stride}_{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, R=4, k=k, stride=stride, pad=pad,
           seed=2300 + i, x_dist="normal")
         for i, (N, Cin, H, W, Cout, k, stride, pad) in enumerate([
             (1, 40, 20, 20, 40, 1, 1, 0), (2, 33, 19, 33, 17, 2, 1, 1), (1, 31, 40, 41, 15, 2, 2, 0), (3, 64, 17, 18, 33, 3, 2, 1),
             (1, 12, 31, 64, 16, 3, 1, 0), (1, 20, 30, 21, 20, 3, 3, 2), (2, 65, 16, 15, 3, 4, 1, 2), (2, 32, 50, 96, 32, 5, 1, 2),
             (1, 96, 16, 16, 24, 5, 1, 2), (1, 97, 17, 29, 31, 5, 2, 2), (2, 8, 64, 64, 32, 7, 1, 3), (1, 70, 16, 28, 16, 7, 2, 3),
             (1, 16, 24, 20, 8, 15, 1, 7), (1, 32, 9, 300, 16, 5, 1, 4)])]


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("cfg", TURNS, ids=[c.name for c in TURNS])
def test_turns(cfg, relu):
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y, yp, _, w_rot = orc.layer_fwd(x, w, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    lay = pu.GpuLayer(cfg, x, w, relu=relu)
    assert lay.plan.kernel_name(0) == "mfma_gemm_scatter" and lay.plan.conv_equivalents(0) == 4
    got, idx = lay.pool_fwd()
    dead = yp <= 0
    if relu:
        sure = np.abs(yp) > 1e-5 * np.abs(yp).max()
        assert np.array_equal((idx == 255)[sure], dead[sure])
        assert _rel(got, np.where(dead, 0, yp)) < _bar(cfg)
        return
    assert _rel(got, yp) < _bar(cfg)
    pu.check_idx(idx, y, orc.rotconv_fwd(np.abs(x), np.abs(w_rot), cfg.stride, cfg.pad), cfg.G, cfg.name)
    again = lay.pool_fwd()
    assert np.array_equal(got, again[0]) and np.array_equal(idx, again[1])
    small = lay.plan.workspace_bytes     # scratch the plan asks for, to the byte
    ws = torch.full((small + 256,), 0xa5, dtype=torch.uint8, device="cuda")
    yp2, idx2 = lay.nan(lay.P), lay.nan(lay.P, torch.uint8)
    rc.rotconv_pool_fwd(lay.plan, lay.x, lay.w, yp2, idx2, ws=ws[:small])
    torch.cuda.synchronize()
    assert np.array_equal(yp2.cpu().numpy(), got) and bool((ws[small:] == 0xa5).all())


@pytest.mark.parametrize("cfg", [TURNS[1], TURNS[8], TURNS[11]], ids=lambda c: c.name)
def test_turns_dyadic(cfg):
    x, w = synth.make_x_dyadic(cfg), synth.make_w_dyadic(cfg)
    _, yp, idx, _ = orc.layer_fwd(x, w, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    got = pu.GpuLayer(cfg, x, w).pool_fwd()
    assert np.array_equal(got[0].astype(np.float64), yp) and np.array_equal(got[1], idx)


ONE = [L(f"o_{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, R=1, seed=2350 + i, x_dist="normal")
       for i, (N, Cin, H, W, Cout) in enumerate([(2, 64, 23, 272, 16), (4, 64, 84, 8, 96), (3, 192, 102, 80, 144), (1, 588, 9, 297, 89),
                                                 (2, 432, 23, 288, 17), (4, 48, 285, 31, 33)])]


@pytest.mark.parametrize("cfg", ONE, ids=[c.name for c in ONE])
def test_single_orientation(cfg):
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    got = lay.fwd().cpu().numpy()
    ref = orc.rotconv_fwd(x, orc.expand_bank(w, 1, None, cfg.mode), 1, 1).reshape(got.shape)
    assert _rel(got, ref) < _bar(cfg)
    placed = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=1)).fwd().cpu().numpy()      # the kernels that place products
    # (both round about as often: 616 layers of 5 to 500 channels 0.99 of the placed form's error in the mean, at most 1.07)
    assert not np.array_equal(got, placed) and _rel(got, ref) < 1.1 * _rel(placed, ref)
    assert torch.equal(lay.fwd(), torch.from_numpy(got).cuda())


@pytest.mark.parametrize("k,stride", [(5, 1), (3, 2), (4, 1)])
def test_values_beyond_the_parts(k, stride):
    """Infinite, huge and tiny operands: as the fp32 sums of the generic kernels have them."""
    cfg = L("beyond", N=1, Cin=40, H=21, W=40, Cout=20, R=4, k=k, stride=stride, pad=k // 2, seed=2380, x_dist="normal")
    x, w = synth.make_x(cfg), synth.make_w(cfg)

    def both(x, w):
        return [pu.GpuLayer(cfg, x, w, options=o).pool_fwd()[0] for o in (dict(), dict(gs=-1))]
    for at in (np.inf, -np.inf, np.nan, 1e30):
        xi = x.copy()
        xi[0, 33, 7, 11] = at
        got, ref = both(xi, w)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        fin = np.isfinite(ref)
        assert np.allclose(got[fin], ref[fin], rtol=1e-4, atol=1e-4 * np.abs(ref[fin & (np.abs(ref) < 1e20)]).max())
    got, ref = both(x * np.float32(1e-22), w * np.float32(1e-14))
    assert _rel(got, ref) < 1e-5


# single orientations with filters of other sizes and strides: even and odd k, with and without centre and remainder of rows, whole and
# with channel shares, channels and filters around a chunk (32) and one or two blocks (16)
ONE_OTHER = [L(f"p{k}_{stride}_{Cin}_{H}x{W}_{Cout}", N=N, Cin=Cin, H=H, W=W, Cout=Cout, R=1, k=k, stride=stride, pad=pad,
               seed=2700 + i, x_dist="normal")
             for i, (N, Cin, H, W, Cout, k, stride, pad) in enumerate([
                 (1, 32, 20, 30, 40, 1, 1, 0), (2, 33, 19, 33, 17, 2, 1, 1), (1, 31, 40, 61, 15, 2, 2, 0), (3, 64, 17, 18, 33, 3, 2, 1),
                 (1, 65, 31, 64, 16, 3, 1, 0), (1, 20, 60, 72, 31, 3, 3, 2), (2, 64, 16, 15, 32, 4, 1, 2), (2, 32, 50, 96, 33, 5, 1, 2),
                 (1, 300, 12, 12, 48, 5, 2, 2), (1, 9, 64, 64, 16, 7, 2, 3), (1, 512, 9, 9, 64, 1, 1, 0), (1, 400, 11, 13, 70, 7, 1, 3),
                 (4, 40, 40, 41, 32, 4, 4, 0), (1, 24, 64, 90, 20, 2, 8, 0)])]


@pytest.mark.parametrize("cfg", ONE_OTHER, ids=[c.name for c in ONE_OTHER])
def test_single_orientation_of_other_filters(cfg):
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    assert lay.plan.kernel_name(0) == "mfma_gemm_scatter"
    got = lay.fwd().cpu().numpy()
    ref = orc.rotconv_fwd(x, orc.expand_bank(w, 1, None, cfg.mode), cfg.stride, cfg.pad).reshape(got.shape)
    assert _rel(got, ref) < _bar(cfg)
    placed = pu.GpuLayer(cfg, x, w, options=dict(gs=1)).fwd().cpu().numpy()
    assert cfg.k == 1 or not np.array_equal(got, placed)       # (1 x 1: the same sums of 32 channels in the same order)
    sure = np.abs(ref) > 1e-5 * np.abs(ref).max()
    for relu in (False, True):
        yp, idx = pu.GpuLayer(cfg, x, w, relu=relu).pool_fwd()
        dead = (ref <= 0) & relu
        assert _rel(yp, np.where(dead, 0, ref)) < _bar(cfg)
        assert np.array_equal(idx[sure], np.where(dead, 255, 0)[sure])


@pytest.mark.parametrize("cfg", [ONE_OTHER[2], ONE_OTHER[6], ONE_OTHER[11]], ids=lambda c: c.name)
def test_single_orientation_of_other_filters_dyadic(cfg):
    x, w = synth.make_x_dyadic(cfg), synth.make_w_dyadic(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    got = lay.fwd().cpu().numpy()
    ref = orc.rotconv_fwd(x, orc.expand_bank(w, 1, None, cfg.mode), cfg.stride, cfg.pad).reshape(got.shape)
    assert np.array_equal(got.astype(np.float64), ref) and np.array_equal(lay.pool_fwd()[0].astype(np.float64), ref)


@pytest.mark.parametrize("k,stride", [(5, 2), (3, 1)])
def test_bf16_tensors(k, stride):
    """A bf16 plan of such a layer widens its tensors and rounds what the fp32 kernels give once: to half a bf16 ulp in the norm."""
    cfg = L("b16", N=2, Cin=40, H=33, W=52, Cout=36, R=4, k=k, stride=stride, pad=0, seed=2750, x_dist="normal")
    r = np.random.default_rng(cfg.seed)
    x, w, g = (pu.round_bf16(a) for a in (synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)))
    plan = rc.Plan.from_config(cfg, dtype=rc.BF16)
    assert [plan.kernel_name(i) for i in range(3)] == ["mfma_gemm_scatter"] * 3 and [plan.conv_equivalents(i) for i in range(3)] == [4] * 3
    xd, wd, gd = (pu.dev(a, torch.bfloat16) for a in (x, w, g))
    yp = torch.full((cfg.N, plan.Cpooled, plan.Ho, plan.Wo), float("nan"), dtype=torch.bfloat16, device="cuda")
    idx = torch.full(yp.shape, 254, dtype=torch.uint8, device="cuda")
    dx, dw = torch.full_like(xd, float("nan")), torch.full(wd.shape, float("nan"), device="cuda")
    y, ref, _, w_rot = orc.layer_fwd(x, w, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    rc.rotconv_pool_fwd(plan, xd, wd, yp, idx)
    pu.check_idx(idx.cpu().numpy(), y, orc.rotconv_fwd(np.abs(x), np.abs(w_rot), cfg.stride, cfg.pad), cfg.G, cfg.name)
    given = r.integers(0, 4, yp.shape).astype(np.uint8)
    rc.rotconv_pool_bwd_data(plan, gd, pu.dev(given), wd, dx)
    rc.rotconv_pool_bwd_weight(plan, xd, gd, pu.dev(given), dw)
    torch.cuda.synchronize()
    rdx, rdw = orc.layer_bwd(x, w, g, given, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)
    assert _rel(yp.float().cpu().numpy(), ref) < 2.0 ** -9 and _rel(dx.float().cpu().numpy(), rdx) < 2.0 ** -9
    assert _rel(dw.cpu().numpy(), rdw) < 5e-7
