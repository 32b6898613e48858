"""The matrix multiply on bf16 parts and the tiled kernels of the multiply + scatter family, at the edges of their tiles:
rows, columns and K-steps around 32, 64 and 128, contractions of one K-step and of many, both sides of the rule that keeps
large products on the fp32 instruction; 32 x 32 pixel tiles of filters from 2 x 2 to 15 x 15 taps, strides to 3, several
banks, incomplete orientation sets, pool groups, images one at a time.

Error bar: within a K-step the matrix instruction cuts six sums per 32 terms, so a sum of K terms is within about
sqrt(6 K / 32) 2^-24 of its norm, and a lone product within 2^-24; n such sums added up one by one are rounded n times at half
their size in the mean: sqrt(1 + 6 K / 32 + n / 2) 2^-24, and twice that is asked for.
"""
import numpy as np
import pytest
import torch

import parity_util as pu
from oracle import rotconv_oracle as orc
from oracle import unet_oracle as uo
from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig


def bar(K, n=0):
    return 2 * 2.0 ** -24 * (1 + 6 * K / 32 + n / 2) ** 0.5


def _rel(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def _err(got, ref, K):
    """Against the norm of sums of K products of unit normals, which a single output may be far below by chance."""
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / max(np.linalg.norm(ref), np.sqrt(K * ref.size)))


@pytest.mark.parametrize("N,Cin,Cout,P", [(1, 1, 9, 1), (2, 31, 33, 63), (1, 32, 64, 64), (3, 33, 65, 65), (2, 64, 31, 129), (1, 97, 130, 31),
                                          (1, 129, 16, 2050), (2, 160, 130, 16389)])      # the last: fp32 instructions
def test_products(N, Cin, Cout, P):
    rng = np.random.default_rng(P)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    x, w, dy = f(N, Cin, 1, P), f(Cout, Cin), f(N, Cout, 1, P)
    y, dx = (torch.full((N, c, 1, P), float("nan"), device="cuda") for c in (Cout, Cin))
    dw = torch.full((Cout, Cin), float("nan"), device="cuda")
    ws = torch.empty(max(256, rc.glue_conv1x1_workspace_bytes(N, Cin, Cout, P)), dtype=torch.uint8, device="cuda")
    xd, wd, gd = pu.dev(x), pu.dev(w), pu.dev(dy)
    rc.glue_conv1x1_fwd(xd, wd, y)
    rc.glue_conv1x1_bwd_data(gd, wd, dx)
    rc.glue_conv1x1_bwd_weight(xd, gd, dw, ws)
    assert _err(y.cpu().numpy(), uo.conv1x1_fwd(x, w), Cin) < bar(Cin)
    dxr, dwr = uo.conv1x1_bwd(x, w, dy)
    assert _err(dx.cpu().numpy(), dxr, Cout) < bar(Cout) and _err(dw.cpu().numpy(), dwr, N * P) < bar(P, N)


@pytest.mark.parametrize("N,Cin,Cout,H,W", [(1, 5, 3, 3, 5), (2, 33, 17, 7, 9), (1, 64, 16, 8, 8), (2, 70, 40, 5, 13)])
def test_pixel_shuffled_products(N, Cin, Cout, H, W):
    rng = np.random.default_rng(H)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    x, w, dy = f(N, Cin, H, W), f(Cin, Cout, 2, 2), f(N, Cout, 2 * H, 2 * W)
    y, dx = torch.full(dy.shape, float("nan"), device="cuda"), torch.full(x.shape, float("nan"), device="cuda")
    dw = torch.full(w.shape, float("nan"), device="cuda")
    ws = torch.empty(max(256, rc.glue_upconv2_workspace_bytes(N, Cin, Cout, H, W)), dtype=torch.uint8, device="cuda")
    xd, wd, gd = pu.dev(x), pu.dev(w), pu.dev(dy)
    rc.glue_upconv2_fwd(xd, wd, y)
    rc.glue_upconv2_bwd_data(gd, wd, dx)
    rc.glue_upconv2_bwd_weight(xd, gd, dw, ws)
    assert _rel(y.cpu().numpy(), uo.upconv2_fwd(x, w)) < bar(Cin)
    dxr, dwr = uo.upconv2_bwd(x, w, dy)
    assert _rel(dx.cpu().numpy(), dxr) < bar(4 * Cout) and _rel(dw.cpu().numpy(), dwr) < bar(H * W, N)


TILES = [
    L("g_k2", N=2, Cin=9, H=33, W=31, Cout=3, R=4, k=2, pad=1, x_dist="normal", seed=1401),
    L("g_k4", N=1, Cin=32, H=32, W=64, Cout=2, R=4, k=4, pad=0, x_dist="normal", seed=1402),
    L("g_k5", N=3, Cin=33, H=34, W=65, Cout=5, R=4, k=5, pad=2, x_dist="normal", seed=1403),
    L("g_k5s2", N=2, Cin=16, H=66, W=35, Cout=4, R=4, k=5, pad=2, stride=2, x_dist="normal", seed=1404),
    L("g_k3s3", N=1, Cin=16, H=40, W=70, Cout=4, R=4, k=3, pad=1, stride=3, x_dist="normal", seed=1405),
    L("g_k7s2", N=1, Cin=8, H=20, W=37, Cout=3, R=8, mode="steerable", k=7, pad=3, stride=2, x_dist="normal", seed=1406),
    L("g_k15", N=1, Cin=4, H=33, W=18, Cout=2, R=4, k=15, pad=7, x_dist="normal", seed=1407),
    L("g_r3", N=1, Cin=8, H=20, W=20, Cout=4, R=3, mode="bilinear", k=5, pad=2, x_dist="normal", seed=1408),
    L("g_g4", N=1, Cin=8, H=20, W=34, Cout=4, R=8, mode="steerable", pool_group=4, k=5, pad=2, x_dist="normal", seed=1409),
]


@pytest.mark.parametrize("chunk", [0, -1])      # all images at once, one at a time
@pytest.mark.parametrize("cfg", TILES, ids=[c.name for c in TILES])
def test_multiply_and_scatter(cfg, chunk):
    x, w, g = synth.make_x(cfg), synth.make_w(cfg), synth.make_g(cfg)
    ref = pu.oracle_layer(cfg, x, w, g)
    lay = pu.GpuLayer(cfg, x, w, options=dict(gs=1, gs_chunk_mb=chunk))
    assert lay.plan.kernel_name(0) == "mfma_gemm_scatter" and lay.plan.bf16_parts(1)
    yp, idx = lay.pool_fwd()
    kk, Q = cfg.k * cfg.k, lay.plan.orientations()[0]
    assert _rel(yp, ref["ypool"]) < bar(cfg.Cin, kk)
    pu.check_idx(idx, ref["y"], ref["abs_terms"], cfg.G, cfg.name)
    assert _rel(lay.fwd().cpu().numpy(), ref["y"].reshape(lay.U)) < bar(cfg.Cin, kk)
    idx = ref["idx"].astype(np.uint8)
    assert _rel(lay.pool_bwd_data(g, idx), ref["dx"]) < bar(kk * Q * cfg.Cout, 4)
    assert _rel(lay.pool_bwd_weight(g, idx), ref["dw"]) < bar(cfg.H * cfg.W, cfg.N + kk)


@pytest.mark.parametrize("k,Cin", [(2, 8), (5, 4), (5, 32), (9, 16), (15, 8)])
def test_forward_has_no_offset(k, Cin):
    """A product of up to 32 channels is one sum, which the matrix instruction cuts: half a unit of its last place, one sign for
    all, would come to k * 1e-8 of the result's norm over the k^2 taps.  Every other tap has the other sign, so one product's
    offset may stay: 3e-8 / k; bar 1.5e-8.  Then the sums over the taps, the same in both forms, are the larger part of the
    error, which is at most that of the fp32 instruction (2 % for the spread of the two)."""
    cfg = L("g_off", N=1, Cin=Cin, H=40, W=40, Cout=8, R=4, k=k, pad=k // 2, x_dist="absnormal", seed=1420 + k)
    x, w = synth.make_x(cfg), synth.make_w(cfg)
    y = orc.rotconv_fwd(x, orc.expand_bank(w, cfg.R, None, cfg.mode), 1, cfg.pad)
    err = []
    for form in (0, -1):
        lay = pu.GpuLayer(cfg, x, w, options=dict(gs=1, bf16_parts=form))
        assert lay.plan.bf16_parts(0) == (form == 0)
        d = lay.fwd().cpu().numpy().astype(np.float64) - y.reshape(lay.U)
        err.append(np.linalg.norm(d))
        assert abs(d.mean()) < 1.5e-8 * np.sqrt(np.mean(y ** 2))
    assert err[0] <= 1.02 * err[1], err


def test_sums_beside_one_the_parts_do_not_hold():
    """... stay bit for bit what they are without it."""
    rng = np.random.default_rng(6)
    N, Cin, Cout, P = 1, 40, 30, 50
    x, w = rng.standard_normal((N, Cin, 1, P)).astype(np.float32), rng.standard_normal((Cout, Cin)).astype(np.float32)

    def run(x):
        y = torch.full((N, Cout, 1, P), float("nan"), device="cuda")
        rc.glue_conv1x1_fwd(pu.dev(x), pu.dev(w), y)
        return y.cpu().numpy()

    clean = run(x)
    for bad in (np.inf, np.nan, 3.4e38, 0.0):
        b = x.copy()
        b[0, 7, 0, 20] = bad
        if bad == 0.0:
            b[0, :, 0, 20] *= 2.0 ** -118
        y = run(b)
        assert np.array_equal(np.delete(y, 20, 3), np.delete(clean, 20, 3)) and not np.array_equal(y[..., 20], clean[..., 20])


def _same(got, ref):
    """Infinities where the reference has them, of its sign, and its values elsewhere."""
    got = np.asarray(got, np.float64)
    fin = np.isfinite(ref)
    assert np.array_equal(got[~fin], ref[~fin]) and np.isfinite(got[fin]).all() and fin.any()
    assert _rel(got[fin], ref[fin]) < bar(234)


@pytest.mark.parametrize("what", ["inf", "large", "tiny"])
def test_values_beyond_the_parts(what):
    """An infinity, 3.4e38 (which no bf16 part holds) and magnitudes of which the parts hold 14 bits: as on the fp32 instruction,
    in tiles with them and in the others, for products of every kind."""
    rng = np.random.default_rng(5)
    N, Cin, Cout, H, W = 2, 70, 20, 9, 13
    f = lambda *s: rng.standard_normal(s).astype(np.float32)

    def hit(a):
        if what == "tiny":
            return np.ldexp(a, -120)
        a.reshape(-1)[a.size // 3] = np.inf if what == "inf" else 3.4e38
        return a

    w = np.clip(f(Cin, Cout, 2, 2), -0.9, 0.9)
    x, dy = f(N, Cin, H, W), f(N, Cout, 2 * H, 2 * W)
    xb, gb = hit(x.copy()), hit(dy.copy())
    y, dx = torch.full(dy.shape, float("nan"), device="cuda"), torch.full(x.shape, float("nan"), device="cuda")
    dw = torch.full(w.shape, float("nan"), device="cuda")
    ws = torch.empty(rc.glue_upconv2_workspace_bytes(N, Cin, Cout, H, W), dtype=torch.uint8, device="cuda")
    small = lambda a: np.clip(a, -0.9, 0.9)
    rc.glue_upconv2_fwd(pu.dev(xb), pu.dev(w), y)
    rc.glue_upconv2_bwd_data(pu.dev(gb), pu.dev(w), dx)
    rc.glue_upconv2_bwd_weight(pu.dev(xb), pu.dev(small(dy)), dw, ws)
    with np.errstate(over="ignore", invalid="ignore"):
        f32 = lambda r: r.astype(np.float32).astype(np.float64) if what != "tiny" else r
        _same(y.cpu().numpy(), f32(uo.upconv2_fwd(xb, w)))
        _same(dx.cpu().numpy(), f32(uo.upconv2_bwd(x, w, gb)[0]))
        _same(dw.cpu().numpy(), f32(uo.upconv2_bwd(xb, w, small(dy))[1]))
    cfg = L("g_big", N=1, Cin=33, H=20, W=22, Cout=4, R=4, k=5, pad=2, x_dist="normal", seed=1430)
    x, w, g = hit(synth.make_x(cfg)), synth.make_w(cfg), np.asarray(synth.make_g(cfg), np.float32)
    idx = rng.integers(0, 4, (1, 4, 20, 22)).astype(np.uint8)
    out = []
    for form in (1, -1):
        lay = pu.GpuLayer(cfg, x, w, options=dict(gs=1, bf16_parts=form))
        out.append((lay.fwd().cpu().numpy(), lay.pool_bwd_data(hit(g.copy()), idx), lay.pool_bwd_weight(small(g), idx)))
    for a, b in zip(*out):
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
        fin = np.isfinite(b)
        assert _rel(a[fin], b[fin].astype(np.float64)) < bar(440, 25)
