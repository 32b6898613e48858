"""A step whose gradients or pixels are NaN throughout: the sums that the parts do not hold are formed again in fp32, at no more
than a bounded multiple of the ordinary time.

Bound: an fp32 multiply-add on the vector ALU with its mask or position takes about four instructions per product of 64 lanes; the six
products of a sum's parts take 6 / 512 of a matrix instruction of 16 clocks: about twenty times the time, with loads that are not
shared thirty.  Kernels of 30 us and more, so that launches do not hide it.
"""
import pytest
import torch

from paper_2512_08888_amd import binding as rc

pytestmark = pytest.mark.gpu

LAYERS = {
    "k5": dict(N=2, Cin=32, H=96, W=96, Cout=32, k=5, pad=2, R=4),
    "k5_strided": dict(N=4, Cin=128, H=128, W=128, Cout=128, k=5, stride=2, pad=2, R=4),
    "k3_strided": dict(N=4, Cin=64, H=56, W=56, Cout=128, k=3, stride=2, pad=1, R=4),
    "one_turn": dict(N=1, Cin=512, H=16, W=16, Cout=128, k=3, pad=1, R=1),
    "first": dict(N=2, Cin=3, H=512, W=512, Cout=64, k=3, pad=1, R=4),
}


def _us(call):
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    call()
    best = 1e30
    for _ in range(3):
        a.record()
        call()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 500)
    return best


@pytest.mark.parametrize("name", list(LAYERS))
def test_a_diverged_step_is_no_hang(name):
    print(f"[case] {name}", flush=True)
    c = dict(LAYERS[name])
    plan = rc.Plan(c.pop("N"), c.pop("Cin"), c.pop("H"), c.pop("W"), c.pop("Cout"), **c)
    d = plan.desc
    torch.manual_seed(1)
    x = torch.randn(d.N, d.Cin, d.H, d.W, device="cuda").relu()
    w = torch.randn(plan.B, d.Cout, d.Cin, d.k, d.k, device="cuda")
    yp = torch.empty(d.N, plan.Cpooled, plan.Ho, plan.Wo, device="cuda")
    idx = torch.empty(yp.shape, dtype=torch.uint8, device="cuda")
    g, dx, dw = torch.randn_like(yp), torch.empty_like(x), torch.empty_like(w)
    rc.rotconv_pool_fwd(plan, x, w, yp, idx)
    other = torch.empty_like(idx)
    times = []
    for bad in (False, True):
        xx, gg = (torch.full_like(t, float("nan")) if bad else t for t in (x, g))
        times.append([_us(lambda: rc.rotconv_pool_fwd(plan, xx, w, yp, other)), _us(lambda: rc.rotconv_pool_bwd_data(plan, gg, idx, w, dx)),
                      _us(lambda: rc.rotconv_pool_bwd_weight(plan, x, gg, idx, dw))])
    assert torch.isnan(dw).any()
    for clean, diverged in zip(*times):
        assert diverged < 30 * clean + 100, times
