"""rotconv_pool_fwd_static takes every layer whose pooled forward fits its scratch by itself, whatever the plan's other calls
need, and gives bit for bit what rotconv_pool_fwd gives."""
import pytest
import torch

from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig

# pooled forwards of 9 to 16 MB beside weight gradients of more than 16 MB, and calls on tensors off their alignment
OWN = [
    (L("pad16", N=1, Cin=23, H=64, W=348, Cout=8, R=1, seed=2201), dict(dtype=rc.BF16), 0),
    (L("pad16_odd", N=13, Cin=30, H=72, W=1, Cout=4, R=1, seed=2202), dict(dtype=rc.BF16), 0),
    (L("native16", N=8, Cin=313, H=100, W=2, Cout=91, R=16, mode="bilinear", seed=2203), dict(dtype=rc.BF16), 0),
    (L("avg", N=1, Cin=26, H=212, W=223, Cout=2, R=4, seed=2204), dict(pool_op="avg"), 0),
    (L("avg_even", N=6, Cin=19, H=43, W=130, Cout=5, R=1, seed=2205), dict(pool_op="avg"), 0),
    (L("avg16", N=8, Cin=30, H=157, W=36, Cout=2, R=2, seed=2206), dict(pool_op="avg", dtype=rc.BF16), 0),
    (L("off", N=4, Cin=19, H=50, W=16, Cout=60, R=1, seed=2207), {}, 1),
    (L("off_k5", N=2, Cin=16, H=20, W=22, Cout=8, R=4, k=5, pad=2, seed=2208), {}, 1),
]


def _both(cfg, over, off):
    plan = rc.Plan.from_config(cfg, **over)
    dt = torch.bfloat16 if over.get("dtype") == rc.BF16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(cfg.seed)

    def t(shape, dtype, fill=None):      # `off` elements off its alignment
        n = 1
        for s in shape:
            n *= s
        v = torch.empty(n + off, dtype=dtype, device="cuda")[off:].view(shape)
        return v.copy_(torch.randn(shape, generator=gen, device="cuda")) if fill is None else v.fill_(fill)

    x = t((cfg.N, cfg.Cin, cfg.H, cfg.W), dt)
    w = t((plan.B, cfg.Cout, cfg.Cin, cfg.k, cfg.k), dt)
    out = []
    for call in (rc.rotconv_pool_fwd, rc.rotconv_pool_fwd_static):
        yp = t((cfg.N, plan.Cpooled, plan.Ho, plan.Wo), dt, float("nan"))
        idx = t(yp.shape, torch.uint8, 254)
        call(plan, x, w, yp, None if over.get("pool_op") == "avg" else idx)
        out.append((yp, idx))
    torch.cuda.synchronize()
    assert torch.isfinite(out[0][0].float()).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("cfg,over,off", OWN, ids=[c.name for c, _, _ in OWN])
def test_own_need(cfg, over, off):
    _both(cfg, over, off)


# layers of which the waves on their own make more parts than the scratch holds: they go through it in slices of filters
# (several blocks, a ragged one, several images), or, where those of sixteen filters do not fit, the contraction stays whole
WHOLE = [
    L("w_r2", N=4, Cin=238, H=10, W=80, Cout=331, R=2, seed=2211),
    L("w_steer", N=6, Cin=378, H=12, W=206, Cout=27, R=8, mode="steerable", pool_group=4, seed=2212),
    L("w_odd", N=13, Cin=230, H=3, W=133, Cout=118, R=4, seed=2214),
    L("w_relu", N=2, Cin=256, H=64, W=64, Cout=128, R=4, seed=2215),
    L("w_one", N=1, Cin=655, H=294, W=80, Cout=46, R=4, seed=2216),
    L("w_r8", N=3, Cin=1207, H=134, W=4, Cout=113, R=8, mode="bilinear", seed=2213),
]


@pytest.mark.parametrize("cfg", WHOLE, ids=[c.name for c in WHOLE])
def test_split_beyond_the_scratch(cfg):
    _both(cfg, dict(relu=cfg.name == "w_relu"), 0)


# averaged plans of few channels on padded rows, up to the scratch's end
AVG_ODD = [
    (L("a_1_64", N=2, Cin=1, H=104, W=205, Cout=64, R=4, seed=2221), dict(pool_op="avg")),
    (L("a_2_36", N=3, Cin=2, H=631, W=37, Cout=36, R=4, seed=2222), dict(pool_op="avg")),
    (L("a_3_30", N=1, Cin=3, H=1230, W=65, Cout=30, R=4, seed=2223), dict(pool_op="avg")),
    (L("a16_2_20", N=1, Cin=2, H=200, W=93, Cout=20, R=4, seed=2224), dict(pool_op="avg", dtype=rc.BF16)),
]


@pytest.mark.parametrize("cfg,over", AVG_ODD, ids=[c.name for c, _ in AVG_ODD])
def test_average_pooling_on_padded_rows(cfg, over):
    _both(cfg, over, 0)


# one contraction whose shares leave room for some of its packed weights only: slices of filter blocks, the last of them ragged, two
# blocks a workgroup; with the workspace all at once
SLICED = [
    (L("s_20_of_71", N=1, Cin=814, H=24, W=19, Cout=1122, R=4, k=1, stride=2, pad=0, seed=2231), {}),
    (L("s_relu_70_of_76", N=1, Cin=667, H=13, W=29, Cout=1212, R=4, k=1, stride=2, pad=0, seed=2232), dict(relu=True)),
    (L("s_one_tile", N=2, Cin=458, H=59, W=3, Cout=1486, R=4, k=1, stride=2, pad=0, seed=2233), {}),
    (L("s_one_turn", N=1, Cin=1026, H=11, W=22, Cout=737, R=1, k=1, pad=0, seed=2234), {}),
]


@pytest.mark.parametrize("cfg,over", SLICED, ids=[c.name for c, _ in SLICED])
def test_one_contraction_in_slices(cfg, over):
    plan = rc.Plan.from_config(cfg, **over)
    assert plan.kernel_name(0) == "mfma_gemm_scatter" and plan.bf16_parts(0) and plan.workspace_bytes > 16 << 20
    _both(cfg, over, 0)
