"""A NaN in the input reaches every pooled value whose window holds it, through the fused ReLU too, on every route of the
pooled forward: the output must not depend on which kernel the dispatch picks."""
import numpy as np
import pytest
import torch

from paper_2512_08888_amd import binding as rc
from paper_2512_08888_amd import synth

pytestmark = pytest.mark.gpu
L = synth.LayerConfig

# (layer, storage, plan options, kernel name, offset of the tensors in elements)
ROUTES = [
    ("parts", L("n_p", N=1, Cin=40, H=9, W=32, Cout=16, R=4, seed=901), "f32", {}, "mfma_p4", 0),
    ("fp32_instructions", L("n_i", N=1, Cin=40, H=9, W=32, Cout=16, R=4, seed=902), "f32", dict(bf16_parts=-1), "mfma_p4", 0),
    ("channel_split", L("n_s", N=1, Cin=256, H=9, W=16, Cout=16, R=4, seed=903), "f32", dict(fwd_csplit=4), "mfma_p4", 0),
    ("folded", L("n_f", N=1, Cin=32, H=9, W=32, Cout=8, R=8, mode="steerable", seed=904), "f32", {}, "mfma_p4", 0),
    ("candidates", L("n_c", N=1, Cin=32, H=9, W=32, Cout=8, R=16, mode="bilinear", seed=905), "f32",
     dict(fwd_base=-1, bf16_parts=-1), "mfma_p4", 0),
    ("base", L("n_b", N=1, Cin=32, H=9, W=32, Cout=8, R=16, mode="bilinear", seed=906), "f32", {}, "mfma_p4_base", 0),
    ("cut_groups", L("n_g", N=1, Cin=32, H=9, W=32, Cout=8, R=4, pool_group=2, seed=907), "f32", {}, "mfma_p4", 0),
    ("odd_rows", L("n_o", N=1, Cin=32, H=9, W=31, Cout=8, R=4, seed=908), "f32", {}, "mfma_p4", 0),
    ("direct", L("n_d", N=1, Cin=3, H=9, W=33, Cout=8, R=4, seed=909), "f32", {}, "valu_direct", 0),
    ("direct_16", L("n_d16", N=1, Cin=3, H=9, W=33, Cout=8, R=16, mode="bilinear", seed=910), "bf16", {}, "valu_direct", 0),
    ("gemm_scatter", L("n_k5", N=1, Cin=32, H=24, W=24, Cout=16, R=4, k=5, pad=2, seed=911), "f32", {}, "mfma_gemm_scatter", 0),
    ("generic", L("n_gen", N=1, Cin=8, H=9, W=32, Cout=8, R=4, k=5, pad=2, seed=912), "f32", dict(gs=-1), "generic", 0),
    ("unaligned", L("n_u", N=1, Cin=16, H=9, W=32, Cout=8, R=4, seed=913), "f32", {}, "mfma_p4", 1),
    ("bf16", L("n_h", N=1, Cin=32, H=9, W=32, Cout=16, R=4, seed=914), "bf16", {}, "mfma_p4_bf16", 0),
    ("bf16_candidates", L("n_h16", N=1, Cin=160, H=9, W=32, Cout=8, R=16, mode="bilinear", seed=915), "bf16", dict(px_fwd=-1),
     "mfma_p4_bf16", 0),
    ("bf16_columns", L("n_px", N=1, Cin=32, H=9, W=32, Cout=8, R=16, mode="bilinear", seed=916), "bf16", {}, "mfma_px_bf16", 0),
]


@pytest.mark.parametrize("cfg,store,options,name,off", [r[1:] for r in ROUTES], ids=[r[0] for r in ROUTES])
def test_nan_reaches_the_pooled_values(cfg, store, options, name, off):
    dt = dict(f32=torch.float32, bf16=torch.bfloat16)[store]
    plan = rc.Plan.from_config(cfg, dtype=dict(f32=rc.F32, bf16=rc.BF16)[store], relu=True, options=options)
    assert plan.kernel_name(0) == name
    w = torch.from_numpy(synth.make_w(cfg)).to(dt).cuda()
    xs = (cfg.N, cfg.Cin, cfg.H, cfg.W)
    ys = (cfg.N, plan.Cpooled, plan.Ho, plan.Wo)

    def run(x):
        xd = torch.zeros(off + x.size, dtype=dt, device="cuda")[off:].view(xs)
        xd.copy_(torch.from_numpy(x).to(dt))
        y = torch.zeros(off + int(np.prod(ys)), dtype=dt, device="cuda")[off:].view(ys)
        idx = torch.full(ys, 254, dtype=torch.uint8, device="cuda")
        rc.rotconv_pool_fwd(plan, xd, w, y, idx)
        return y.float().cpu().numpy(), idx.cpu().numpy()

    x = synth.make_x(cfg)
    clean, cidx = run(x)
    assert np.isfinite(clean).all() and (clean >= 0).all()
    x[0, 2, 4, 10] = np.nan
    y, idx = run(x)
    reached = np.zeros((plan.Ho, plan.Wo), bool)
    r = cfg.k // 2
    reached[4 - r:5 + r, 10 - r:11 + r] = True
    assert np.isnan(y[0][:, reached]).all()
    assert (idx[0][:, reached] < cfg.R).all()             # some orientation, not the dead element's 255
    assert np.array_equal(y[0][:, ~reached], clean[0][:, ~reached])
    assert np.array_equal(idx[0][:, ~reached], cidx[0][:, ~reached])
