"""The fp32 kernels that multiply bf16 parts of their operands: edges of their tiles and of their dispatch against the
oracle, both forms of the products (plan option bf16_parts), lone products and precision against the fp32 instructions,
exact scaling by powers of two (down to where a value's parts are bf16 numbers) and what is lost below, non-finite inputs,
channel splits, and what the static scratch takes.

Error bar where none is given: a 32-term instruction cuts six sums per 32 channels, the last by up to an ulp of its own
size, so a sum over K channels and nine taps is within about sqrt(6 K / 32) * 2^-24 of its value in norm; the bar is 1e-6,
four times that for the deepest case (K = 600).
"""
import numpy as np
import pytest
import torch

import parity_util as pu
from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth
from oracle import rotconv_oracle as orc

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


FWD = [
    L("s_c5", N=2, Cin=5, H=6, W=10, Cout=17, R=4, x_dist="normal", seed=811),                # ragged chunk, second filter block
    L("s_c33", N=1, Cin=33, H=9, W=34, Cout=16, R=4, x_dist="normal", seed=812),              # a chunk with one channel
    L("s_c160", N=1, Cin=160, H=5, W=32, Cout=16, R=1, x_dist="absnormal", seed=813),         # the largest resident block
    L("s_c161", N=1, Cin=161, H=5, W=32, Cout=20, R=4, x_dist="absnormal", seed=814),         # the smallest streamed block
    L("s_c200m", N=1, Cin=200, H=4, W=30, Cout=16, R=4, x_dist="normal", seed=815),           # streamed, rows with masks
    L("s_fold", N=1, Cin=192, H=4, W=32, Cout=8, R=8, mode="steerable", x_dist="normal", seed=816),   # folded banks, streamed
    L("s_c600", N=1, Cin=600, H=4, W=8, Cout=16, R=4, x_dist="absnormal", seed=817),
]


@pytest.mark.parametrize("csplit", [1, 3])
@pytest.mark.parametrize("cfg", FWD, ids=[c.name for c in FWD])
def test_forward_edges(cfg, csplit):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=csplit))
    yp, idx = lay.pool_fwd()
    assert _rel(yp, ref["ypool"]) < 1e-6
    pu.check_idx(idx, ref["y"], ref["abs_terms"], cfg.G, cfg.name)
    yu = lay.nan(lay.U)
    rc.rotconv_fwd(lay.plan, lay.x, lay.w, yu)
    assert _rel(yu.cpu().numpy(), ref["y"].reshape(yu.shape)) < 1e-6


def test_forward_scales_by_powers_of_two():
    cfg = L("s_scale", N=1, Cin=40, H=6, W=32, Cout=16, R=4, x_dist="normal", seed=821)
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y0, i0 = pu.GpuLayer(cfg, x, w).pool_fwd()
    for ex, ew in ((60, 0), (-60, 0), (50, 30), (-40, -30)):
        y, i = pu.GpuLayer(cfg, np.ldexp(x, ex), np.ldexp(w, ew)).pool_fwd()
        assert np.array_equal(y, np.ldexp(y0, ex + ew)) and np.array_equal(i, i0)


def test_forward_shows_non_finite_inputs():
    """An infinite or NaN input makes every pooled value it reaches non-finite, through the fused ReLU too."""
    cfg = L("s_inf", N=1, Cin=16, H=9, W=32, Cout=16, R=4, x_dist="absnormal", seed=822)
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    for bad in (np.inf, -np.inf, np.nan):
        xb = x.copy()
        xb[0, 3, 4, 10] = bad
        for relu in (False, True):
            yp, _ = pu.GpuLayer(cfg, xb, w, relu=relu).pool_fwd()
            reached = np.zeros((9, 32), bool)
            reached[3:6, 9:12] = True
            assert not np.isfinite(yp[0][:, reached]).any() and np.isfinite(yp[0][:, ~reached]).all()


def test_static_scratch_takes_a_slice_of_the_banks_at_a_time():
    cfg = L("s_slice", N=1, Cin=640, H=6, W=32, Cout=640, R=4, x_dist="absnormal", seed=823)     # 14.7 MB at 4 bytes a weight
    plan = rc.Plan.from_config(cfg)
    x, w = pu.dev(synth.make_x(cfg)), pu.dev(synth.make_w(cfg))
    out = []
    for call in (rc.rotconv_pool_fwd, rc.rotconv_pool_fwd_static):
        yp = torch.full((1, plan.Cpooled, 6, 32), float("nan"), device="cuda")
        idx = torch.full(yp.shape, 254, dtype=torch.uint8, device="cuda")
        call(plan, x, w, yp, idx)
        out.append((yp, idx))
    torch.cuda.synchronize()
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0], out[1][0])


# channel blocks of 32 in workgroups of two or four, filter blocks of 32, strips of 16 pixels, rows in pairs
WGRAD = [
    L("w_c33", N=1, Cin=33, H=5, W=4, Cout=31, R=4, x_dist="normal", seed=831),               # one strip, mostly absent
    L("w_c64", N=2, Cin=64, H=7, W=16, Cout=33, R=4, x_dist="normal", seed=832),              # the largest block of two
    L("w_c65", N=1, Cin=65, H=8, W=20, Cout=32, R=1, x_dist="normal", seed=833),              # the smallest block of four
    L("w_c129", N=1, Cin=129, H=1, W=36, Cout=16, R=4, x_dist="normal", seed=834),            # three blocks of two, one row
    L("w_c193", N=3, Cin=193, H=2, W=12, Cout=5, R=2, x_dist="normal", seed=835),             # two blocks of four
    L("w_units", N=8, Cin=40, H=128, W=160, Cout=40, R=4, x_dist="absnormal", seed=836),           # workgroups with several units
    L("w_g2", N=2, Cin=72, H=9, W=16, Cout=24, R=8, mode="steerable", pool_group=4, x_dist="normal", seed=837),
]


@pytest.mark.parametrize("cfg", WGRAD, ids=[c.name for c in WGRAD])
def test_weight_gradient_edges(cfg):
    """A third of the winners are the byte 255, which no orientation has (the fused ReLU's zero): their gradient is
    dropped.  Bar: a sum of n products that is rounded after every 16 of them is within about sqrt(n / 32) * 2^-25 of its
    value in norm, 2.4e-7 for the 1280 of a workgroup's share here; 5e-7.  An offset of the same sign in each of the
    matrix instructions would show above it in w_units."""
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, x, w)
    rng = np.random.default_rng(cfg.seed)
    idx = rng.integers(0, cfg.G, lay.P).astype(np.uint8)
    off = rng.random(lay.P) < 1 / 3
    ref = orc.layer_bwd(x, w, np.where(off, 0, g), idx, cfg.R, None, cfg.mode, cfg.stride, cfg.pad, cfg.G)[1]
    assert _rel(lay.pool_bwd_weight(g, np.where(off, 255, idx).astype(np.uint8)), ref) < 5e-7


# 30-slot tiles over padded rows laid end to end, K-steps of 16 filters, blocks of 32 channels; at the sizes from which the
# kernel is taken
DGRAD = [
    L("d_c33", N=2, Cin=33, H=127, W=126, Cout=72, R=4, x_dist="normal", seed=841),           # the last K-step starts early
    L("d_f9", N=4, Cin=64, H=200, W=202, Cout=9, R=4, x_dist="normal", seed=842),             # the lane halves' filters overlap
    L("d_f5", N=4, Cin=64, H=250, W=248, Cout=5, R=1, x_dist="normal", seed=843),             # ... and coincide
    L("d_w4", N=4, Cin=128, H=848, W=4, Cout=128, R=4, x_dist="normal", seed=844),            # six-slot rows, shared out
    L("d_ks", N=4, Cin=250, H=28, W=30, Cout=300, R=4, x_dist="normal", seed=845),            # shared out, ragged both ways
    L("d_odd", N=2, Cin=48, H=181, W=181, Cout=48, R=2, x_dist="normal", seed=846),           # an odd width
    L("d_g2", N=2, Cin=72, H=101, W=104, Cout=40, R=8, mode="steerable", pool_group=4, x_dist="normal", seed=847),
]


@pytest.mark.parametrize("cfg", DGRAD, ids=[c.name for c in DGRAD])
def test_input_gradient_edges(cfg):
    """Bar as for the forward pass: six sums per 16 filters and tap, each rounded to half an ulp."""
    w, g = synth.make_w(cfg), synth.make_g(cfg)
    lay = pu.GpuLayer(cfg, np.zeros((cfg.N, cfg.Cin, cfg.H, cfg.W), np.float32), w)
    rng = np.random.default_rng(cfg.seed)
    idx = rng.integers(0, cfg.G, lay.P).astype(np.uint8)
    off = rng.random(lay.P) < 1 / 3
    dy = orc.orient_maxpool_bwd(np.where(off, 0, g), idx, cfg.R, cfg.G)
    ref = orc.rotconv_bwd_data(dy, orc.expand_bank(w, cfg.R, None, cfg.mode), cfg.H, cfg.W, cfg.stride, cfg.pad)
    assert _rel(lay.pool_bwd_data(g, np.where(off, 255, idx).astype(np.uint8)), ref) < 1e-6


# the smallest layers, which the automatic choice leaves to the fp32 instructions in one pass or another, and streamed and
# masked instances of both forms of the forward
EITHER = [
    L("e_1", N=1, Cin=5, H=1, W=4, Cout=1, R=4, x_dist="normal", seed=851),
    L("e_r1", N=2, Cin=9, H=3, W=8, Cout=17, R=1, x_dist="normal", seed=852),
    L("e_c32", N=1, Cin=32, H=5, W=32, Cout=16, R=4, x_dist="normal", seed=853),
    L("e_c33", N=2, Cin=33, H=6, W=36, Cout=20, R=4, x_dist="normal", seed=854),
    L("e_c225", N=1, Cin=225, H=3, W=64, Cout=16, R=2, x_dist="normal", seed=855),            # streamed in both forms
    L("e_c260m", N=1, Cin=260, H=4, W=44, Cout=18, R=4, x_dist="normal", seed=856),           # ... rows with masks
    L("e_g4", N=1, Cin=40, H=7, W=20, Cout=8, R=8, mode="steerable", pool_group=4, x_dist="normal", seed=857),
    L("e_fold", N=1, Cin=64, H=7, W=32, Cout=8, R=8, mode="steerable", x_dist="normal", seed=858),
]


@pytest.mark.parametrize("form", [1, -1])
@pytest.mark.parametrize("cfg", EITHER, ids=[c.name for c in EITHER])
def test_both_forms_at_the_smallest_sizes(cfg, form):
    """Plan option bf16_parts; bar as above."""
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    for csplit in (1, 0):
        lay = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=csplit, bf16_parts=form))
        assert [lay.plan.bf16_parts(i) for i in range(3)] == [form > 0] * 3
        yp, idx = lay.pool_fwd()
        assert _rel(yp, ref["ypool"]) < 1e-6
        pu.check_idx(idx, ref["y"], ref["abs_terms"], cfg.G, cfg.name)
        assert _rel(lay.fwd().cpu().numpy(), ref["y"].reshape(lay.U)) < 1e-6
    assert _rel(lay.pool_bwd_weight(g, ref["idx"]), ref["dw"]) < 1e-6
    assert _rel(lay.pool_bwd_data(g, ref["idx"]), ref["dx"]) < 1e-6


def _hard(rng, shape):
    """Values whose low parts are as large as they get, next to random ones; any sign, seven binades."""
    low = np.array([0xffff, 0x1ffff, 0x7fbf, 0x7fff, 0x8000, 0x8041, 0x7fffff, 0x7f7fbf], np.uint32)
    bits = np.where(rng.random(shape) < 0.7, rng.choice(low, shape), rng.integers(0, 1 << 23, shape)).astype(np.uint32)
    v = (bits | np.uint32(0x3f800000)).view(np.float32)
    return np.ldexp(v, rng.integers(-3, 4, shape)) * rng.choice(np.float32([-1, 1]), shape)


def _lone_product_error(got, ref):
    """Largest error of a value over the value itself (zeros have to be zeros)."""
    got = np.asarray(got, np.float64)
    assert np.array_equal(got[ref == 0], ref[ref == 0]) and np.count_nonzero(ref) > 500
    return float(np.max(np.abs(got - ref)[ref != 0] / np.abs(ref)[ref != 0]))


def test_lone_products():
    """Sums of which only one term is not zero, so that nothing averages out.  The three products of parts left out are at
    most 2^-24 of the product, and the sum of the other six is cut to 24 bits (less than 2^-23): bar 1.02 (2^-24 + 2^-23)."""
    bar = 1.02 * (2.0 ** -24 + 2.0 ** -23)
    rng = np.random.default_rng(861)
    cfg = L("s_lone", N=2, Cin=40, H=12, W=24, Cout=24, R=4, x_dist="normal", seed=861)
    spots = np.zeros((12, 24), bool)
    spots[1::3, 1::3] = True                                   # no window holds two of them
    one = np.zeros((cfg.N, cfg.Cin, 12, 24), bool)             # ... each in one channel
    ch = rng.integers(0, cfg.Cin, (cfg.N, 12, 24))
    np.put_along_axis(one, ch[:, None], spots[None, None].repeat(cfg.N, 0), 1)
    x, w = np.where(one, _hard(rng, one.shape), 0).astype(np.float32), _hard(rng, (1, cfg.Cout, cfg.Cin, 3, 3))
    lay = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=1))
    y = orc.rotconv_fwd(x, orc.expand_bank(w, cfg.R, None, cfg.mode), 1, 1)
    assert _lone_product_error(lay.fwd().cpu().numpy(), y.reshape(lay.U)) < bar

    one = np.zeros(lay.P, bool)                                # one filter per spot: lone products in the input gradient
    co = rng.integers(0, cfg.Cout, (cfg.N, 12, 24))
    np.put_along_axis(one, co[:, None], spots[None, None].repeat(cfg.N, 0), 1)
    g, idx = np.where(one, _hard(rng, lay.P), 0).astype(np.float32), rng.integers(0, 4, lay.P).astype(np.uint8)
    dy = orc.orient_maxpool_bwd(g, idx, cfg.R, cfg.G)
    dx = orc.rotconv_bwd_data(dy, orc.expand_bank(w, cfg.R, None, cfg.mode), 12, 24, 1, 1)
    assert _lone_product_error(lay.pool_bwd_data(g, idx), dx) < bar

    g = np.zeros(lay.P, np.float32)                            # one pixel per filter: lone products in the weight gradient
    for c in range(cfg.Cout):
        g[rng.integers(cfg.N), c, rng.integers(12), rng.integers(24)] = _hard(rng, ())
    x = _hard(rng, x.shape)
    lay = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=1))
    dw = orc.layer_bwd(x, w, g, idx, cfg.R, None, cfg.mode, 1, 1, cfg.G)[1]
    assert _lone_product_error(lay.pool_bwd_weight(g, idx), dw) < bar


def test_forward_has_no_offset():
    """The matrix instruction cuts its sums, one sign for all: half a unit of the last place of a chunk's sum, in each of the
    chunks x taps, would come to about 1.2e-7 of the result's norm here (2048 channels).  Four of the nine taps' products
    are formed with the other sign, so a ninth of it may stay: 1.4e-8, bar 3e-8."""
    cfg = L("s_deep", N=1, Cin=2048, H=8, W=32, Cout=32, R=4, x_dist="absnormal", seed=871)
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y = orc.rotconv_fwd(x, orc.expand_bank(w, cfg.R, None, cfg.mode), 1, 1)
    for csplit in (1, 16):
        lay = pu.GpuLayer(cfg, x, w, options=dict(fwd_csplit=csplit, bf16_parts=1))
        err = lay.fwd().cpu().numpy().astype(np.float64) - y.reshape(lay.U)
        assert abs(float(err.mean())) < 3e-8 * float(np.sqrt(np.mean(y ** 2)))


PRECISE = [
    L("p_plain", N=1, Cin=512, H=16, W=16, Cout=128, R=1, x_dist="absnormal", seed=872),      # sixteen parts of one chunk
    L("p_deep", N=1, Cin=1024, H=16, W=16, Cout=64, R=1, x_dist="absnormal", seed=873),
    L("p_few", N=1, Cin=48, H=40, W=40, Cout=24, R=4, x_dist="absnormal", seed=874),
]


@pytest.mark.parametrize("cfg", PRECISE, ids=[c.name for c in PRECISE])
def test_forward_is_no_less_precise_than_fp32_instructions(cfg):
    """Against 64 bits, on the same inputs."""
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y = orc.rotconv_fwd(x, orc.expand_bank(w, cfg.R, None, cfg.mode), 1, 1)
    err = []
    for form in (1, -1):
        lay = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=form))
        err.append(_rel(lay.fwd().cpu().numpy(), y.reshape(lay.U)))
    assert err[0] <= err[1], err


@pytest.mark.parametrize("cout", [9, 16, 24, 31, 32, 40, 200, 1024, 1025])
def test_gradients_are_no_less_precise_than_fp32_instructions(cout):
    """Against 64 bits, on the same inputs; the contraction of the input gradient runs over the filters."""
    cfg = L(f"p_g{cout}", N=2, Cin=48, H=24, W=36, Cout=cout, R=4, x_dist="absnormal", seed=875 + cout)
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    idx = np.random.default_rng(cfg.seed).integers(0, 4, (cfg.N, cout, cfg.H, cfg.W)).astype(np.uint8)
    dx, dw = orc.layer_bwd(x, w, g, idx, cfg.R, None, cfg.mode, 1, 1, cfg.G)
    err = []
    for form in (1, -1):
        lay = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=form))
        err.append((_rel(lay.pool_bwd_data(g, idx), dx), _rel(lay.pool_bwd_weight(g, idx), dw)))
    assert err[0][0] <= err[1][0] and err[0][1] <= err[1][1], err


@pytest.mark.parametrize("form", [1, -1])
@pytest.mark.parametrize("parts", [(256, 256), (192, 192, 128), (128, 128, 128, 128)], ids=lambda p: str(len(p)))
def test_channel_split_has_the_parts_asked_for(parts, form):
    """fwd_csplit = n on 512 channels, of which a filter block's share is streamed (8, 6 chunks of 32) or stays in LDS (4):
    the result is, bit for bit, the ordered sum of the layer's n parts computed as layers of their own."""
    cfg = L("s_parts", N=2, Cin=512, H=5, W=24, Cout=20, R=4, x_dist="normal", seed=881)
    x, w = synth.make_x(cfg), synth.make_w(cfg)

    def fwd(a, b, split):
        c = L("s_part", N=2, Cin=b - a, H=5, W=24, Cout=20, R=4, x_dist="normal", seed=881)
        lay = pu.GpuLayer(c, x[:, a:b], w[:, :, a:b], options=dict(fwd_csplit=split, bf16_parts=form))
        return lay.fwd().cpu().numpy()

    want, at = 0, 0
    for n in parts:
        want, at = want + fwd(at, at + n, 1), at + n
    assert np.array_equal(fwd(0, 512, len(parts)), want)


STATIC = [
    L("t_smaller", N=7, Cin=1504, H=9, W=8, Cout=128, R=4, seed=891),                   # taken with a smaller split
    L("t_whole", N=7, Cin=128, H=36, W=8, Cout=144, R=4, seed=892),                     # not split: four chunks
    L("t_one_block", N=1, Cin=1300, H=4, W=8, Cout=16, R=64, mode="steerable", seed=893),     # 16 banks of one filter block
    L("t_refused", N=4, Cin=512, H=32, W=32, Cout=128, R=4, seed=894),                  # four parts of 8 MB
]


@pytest.mark.parametrize("cfg", STATIC, ids=[c.name for c in STATIC])
def test_static_scratch_takes_the_same_kernels_or_refuses(cfg):
    """The call without a workspace never changes the order of the sums to make a layer fit."""
    plan = rc.Plan.from_config(cfg)
    gen = torch.Generator(device="cuda").manual_seed(cfg.seed)
    x = torch.randn((cfg.N, cfg.Cin, cfg.H, cfg.W), generator=gen, device="cuda")
    w = torch.randn((plan.B, cfg.Cout, cfg.Cin, 3, 3), generator=gen, device="cuda")

    def run(call):
        yp = torch.full((cfg.N, plan.Cpooled, cfg.H, cfg.W), float("nan"), device="cuda")
        idx = torch.full(yp.shape, 254, dtype=torch.uint8, device="cuda")
        call(plan, x, w, yp, idx)
        return yp, idx

    want = run(rc.rotconv_pool_fwd)
    if cfg.name == "t_refused":
        with pytest.raises(rc.RotconvError) as e:
            run(rc.rotconv_pool_fwd_static)
        assert e.value.status == rc.ERR_WORKSPACE
    else:
        got = run(rc.rotconv_pool_fwd_static)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_small_magnitudes():
    """From 2^-110 up the parts hold a float whole: results scale with it bit for bit.  Below, a value is held to 2^-134,
    half a unit of the smallest bf16 number; on the fp32 instructions (bf16_parts = -1) it is not."""
    cfg = L("s_tiny", N=1, Cin=40, H=6, W=32, Cout=24, R=4, x_dist="normal", seed=898)
    rng = np.random.default_rng(cfg.seed)

    def unit(*shape):
        return (rng.uniform(1, 2, shape) * rng.choice([-1, 1], shape)).astype(np.float32)

    x, w = unit(cfg.N, cfg.Cin, cfg.H, cfg.W), unit(1, cfg.Cout, cfg.Cin, 3, 3)
    g, idx = unit(cfg.N, cfg.Cout, cfg.H, cfg.W), rng.integers(0, 4, (cfg.N, cfg.Cout, cfg.H, cfg.W)).astype(np.uint8)

    def passes(e, form):
        lay = pu.GpuLayer(cfg, np.ldexp(x, e), w, options=dict(bf16_parts=form))
        gone = pu.GpuLayer(cfg, x, w, options=dict(bf16_parts=form)).pool_bwd_data(np.ldexp(g, e), idx)
        return lay.fwd().cpu().numpy(), lay.pool_bwd_weight(g, idx), gone

    whole = passes(0, 1)
    for e in (-60, -110):
        assert all(np.array_equal(a, np.ldexp(b, e)) for a, b in zip(passes(e, 1), whole))
    # at most 9 * 40 (forward), 192 (weight gradient), 9 * 24 products of a value held to 2^-134 and one below 2, in units of 2^-120
    for a, b, n in zip(passes(-120, 1), whole, (360, 192, 216)):
        err = np.abs(np.ldexp(a.astype(np.float64), 120) - b)
        assert 0 < err.max() < n * 2 * 2.0 ** (120 - 134) + 1e-6 * np.abs(b).max()
    assert all(_rel(np.ldexp(a.astype(np.float64), 120), b.astype(np.float64)) < 1e-6
               for a, b in zip(passes(-120, -1), whole))
