"""Which fp32 passes multiply bf16 parts of their operands (host logic only), and that the GPU cases written for those
kernels are taken by them."""
import pytest

import test_gpu_split as gs
from paper_2512_08888_amd import binding as rc


def parts(*a, **k):
    p = rc.Plan(*a, **k)
    return [p.bf16_parts(i) for i in range(3)]


def test_selection():
    assert parts(8, 64, 256, 256, 64) == [True] * 3
    assert parts(8, 64, 256, 256, 64, options=dict(bf16_parts=-1)) == [False] * 3
    # short contractions keep the fp32 input gradient, up to 32 channels the fp32 weight gradient
    assert parts(1, 40, 32, 32, 16) == [True, False, True]
    assert parts(1, 16, 32, 32, 16) == [True, False, False]
    assert parts(1, 16, 32, 32, 16, options=dict(bf16_parts=1)) == [True] * 3
    # other turns: the forward on base products, while the table gradients stay with fp32 instructions
    assert parts(4, 128, 128, 128, 128, R=16, mode="bilinear") == [True, False, False]
    assert parts(4, 128, 128, 128, 128, R=16, mode="bilinear", options=dict(bf16_parts=-1)) == [False] * 3
    assert parts(4, 128, 128, 128, 128, R=16, mode="bilinear", options=dict(fwd_base=-1)) == [True, False, False]
    # a first layer: unless the vector ALU is asked for, by form, by band or by what it alone takes
    assert parts(2, 3, 512, 512, 64)[::2] == [True, True]
    for other in (dict(options=dict(bf16_parts=-1)), dict(options=dict(direct_ty=1)), dict(dtype=rc.BF16), dict(R=16, mode="bilinear")):
        assert parts(2, 3, 512, 512, 64, **other)[::2] == [False, False], other
    assert parts(2, 3, 512, 510, 64)[::2] == [False, True] and parts(2, 4, 512, 512, 64)[::2] == [False, True]
    assert not parts(2, 3, 512, 3, 64)[2]
    assert parts(8, 64, 256, 256, 64, dtype=rc.BF16) == [False] * 3
    # other filters: one contraction always, in each pass that runs as one
    assert parts(2, 32, 96, 96, 32, k=5, pad=2) == [True] * 3
    assert parts(2, 32, 96, 96, 32, k=5, pad=2, options=dict(bf16_parts=-1)) == [False] * 3
    assert parts(6, 53, 188, 58, 25, k=5, stride=2, pad=2) == [True] * 3
    # matrix multiply + scatter: products of fewer than 512 tiles of 128 x 128 (forward 7 x 72 an image, input gradient 72,
    # weight gradient 7 in 36 parts)
    placed = dict(k=5, pad=2, options=dict(gs=1))
    assert parts(2, 32, 96, 96, 32, **placed) == [False, True, True]
    assert parts(1, 32, 96, 96, 32, **placed) == [True] * 3
    assert parts(2, 32, 96, 96, 32, k=5, pad=2, options=dict(bf16_parts=1)) == [True] * 3
    assert parts(3, 40, 101, 75, 24, R=8, mode="steerable", pool_group=4)[0]            # odd rows: the padded plan's
    assert parts(8, 64, 256, 256, 64, pool_op="avg") == [True] * 3                      # the averaged bank's plan
    # nor do few filters or single rows take it where the partial sums are most of the work
    assert [parts(5, 393, 12, 20, c)[2] for c in (3, 16, 17, 64)] == [False, False, True, True]
    assert [parts(5, 415, h, 96, 43)[2] for h in (1, 2)] == [False, True]
    assert [parts(5, c, 12, 20, 3)[2] for c in (128, 393)] == [True, False]
    assert parts(5, 393, 12, 20, 3, options=dict(bf16_parts=1))[2]
    # an image of the pooled gradient of 2^32 - 8 bytes: positions outside it have the offset 2^32 - 16, which would lie inside
    assert parts(1, 8, 1103, 4178, 233, R=1, options=dict(bf16_parts=1))[1] is False
    assert parts(1, 8, 1103, 4176, 233, R=1, options=dict(bf16_parts=1))[1] is True


@pytest.mark.parametrize("cfgs,which", [(gs.FWD, 0), (gs.WGRAD, 2), (gs.DGRAD, 1)], ids=["forward", "weight", "input"])
def test_edge_cases_reach_the_kernels_they_are_for(cfgs, which):
    for cfg in cfgs:
        assert rc.Plan.from_config(cfg).bf16_parts(which), cfg.name


def test_odd_rows_of_pool_groups_over_several_banks_are_padded():
    """The folded forward has no instances for odd rows: its plans copy them to padded rows, whose workspace shows."""
    for kw in (dict(R=8, mode="steerable"), dict(R=16, mode="bilinear")):
        for opt in (None, dict(fwd_base=-1)):
            odd, even = (rc.Plan(2, 24, 40, W, 12, options=opt, **kw) for W in (39, 40))
            assert odd.kernel_name(0) == even.kernel_name(0)
            assert odd.workspace_bytes > even.workspace_bytes


def test_executed_work_of_one_contraction():
    """Four products where the turns are rows of one contraction, one where they share a tap's product."""
    work = lambda *a, **k: [rc.Plan(*a, **k).conv_equivalents(i) for i in range(3)]
    assert work(2, 32, 96, 96, 32, k=5, pad=2) == [4, 4, 4]
    assert work(2, 32, 96, 96, 32, k=5, pad=2, options=dict(gs=1)) == [1, 1, 1]
    assert work(4, 200, 96, 96, 200, k=5, pad=2) == [1, 1, 1]                # deep layers: products placed, gradients routed
    assert work(6, 53, 188, 58, 25, k=5, stride=2, pad=2) == [4, 4, 4]
    assert work(2, 3, 512, 512, 64)[::2] == [4, 4]
    assert work(2, 3, 512, 512, 64, options=dict(bf16_parts=-1))[::2] == [1, 1]
    assert work(2, 32, 96, 96, 32, R=1, k=5, pad=2)[0] == 1


def test_strides_that_one_contraction_takes():
    """Strides up to 8 (each remainder of a pixel is a launch dimension), the forward up to four times the filter."""
    taken = lambda k, stride: [rc.Plan(4, 64, 40 * stride, 30 * stride, 128, k=k, stride=stride, pad=k // 2).conv_equivalents(i) == 4 for i in (0, 1)]
    assert taken(3, 6) == [True, True] and taken(2, 8) == [True, True] and taken(1, 4) == [True, True]
    assert taken(3, 8) == [False, True]                     # no tile of 64 outputs whose pixels fit LDS
    assert taken(1, 5) == [False, True] and taken(3, 9) == [False, False]
    assert [rc.Plan(4, 64, 600, 600, 128, k=3, stride=300, pad=1).conv_equivalents(i) for i in range(3)] == [1, 1, 1]


def test_one_contraction_keeps_to_the_scratch_that_the_caller_bounds():
    """gs_chunk_mb: beside what the placed products take, the packed weights (six bytes each, padded to 32) and a MiB for the weight
    gradient's partial sums."""""
    for N, Cin, H, W, Cout, k, stride in ((3, 8, 34, 12, 14, 7, 1), (4, 43, 9, 17, 20, 7, 2), (8, 60, 30, 40, 40, 7, 1), (6, 64, 24, 24, 300, 5, 1), (4, 64, 28, 28, 64, 5, 2)):
        ws = [rc.Plan(N, Cin, H, W, Cout, k=k, stride=stride, pad=k // 2, options=dict(gs_chunk_mb=-1, gs=gs)).workspace_bytes for gs in (0, 1)]
        pad32 = lambda v: (v + 31) // 32 * 32
        assert ws[0] <= ws[1] + 6 * pad32(Cin) * pad32(Cout) * k * k + (1 << 20)


def one_contraction(which):
    """Does pass `which` of a pooled layer of four turns run as one contraction (which multiplies parts whatever the tiles)?"""
    return lambda N, Cin, H, W, Cout, k, stride=1: rc.Plan(N, Cin, H, W, Cout, k=k, stride=stride, pad=k // 2 if k > 1 else 0).conv_equivalents(which) == 4


def test_forward_of_few_filters_and_sparse_pixels():
    """On both sides of its lines, which follow measured times."""
    taken = one_contraction(0)
    assert not taken(7, 66, 238, 240, 1, 5) and not taken(6, 94, 244, 257, 2, 4) and not taken(8, 84, 195, 106, 5, 5)
    assert taken(7, 66, 20, 20, 1, 5) and taken(6, 94, 60, 60, 2, 4) and taken(8, 84, 195, 106, 9, 5)
    assert taken(7, 66, 238, 240, 1, 5, stride=2)
    assert not taken(3, 114, 212, 33, 50, 1, stride=3) and not taken(7, 192, 152, 90, 11, 2, stride=3)
    assert taken(3, 64, 212, 33, 50, 1, stride=3) and taken(3, 114, 40, 33, 50, 1, stride=3) and taken(3, 114, 212, 33, 50, 1, stride=2)
    # a single orientation: fewer tiles of products than 512 are on parts either way
    one = lambda *a: rc.Plan(*a, R=1, k=7, pad=3).bf16_parts(0)
    assert not one(7, 39, 179, 105, 1) and one(7, 39, 179, 105, 8) and one(4, 39, 90, 105, 1)


def test_input_gradient_of_few_filters_and_sparse_pixels():
    taken = one_contraction(1)
    assert [taken(4, 59, 198, 105, c, 5) for c in (1, 3, 7, 8, 16)] == [False, False, False, True, True]
    assert [taken(4, 59, 98, 105, c, 2) for c in (1, 8, 9)] == [False, False, True]
    assert [taken(1, 30, 30, 30, c, 7, stride=2) for c in (4, 7, 8)] == [False, False, True]
    assert [taken(8, 235, 180, 81, c, 1, stride=4) for c in (14, 24, 25)] == [False, False, True]
    assert taken(1, 235, 180, 81, 14, 1, stride=4) and taken(8, 235, 180, 81, 14, 2, stride=2)


def test_weight_gradient_of_few_filters():
    taken = one_contraction(2)
    assert not taken(4, 59, 198, 105, 3, 5) and not taken(4, 112, 292, 170, 1, 7, stride=2) and not taken(8, 3, 50, 146, 1, 2)
    assert taken(4, 59, 40, 105, 3, 5) and taken(4, 59, 198, 105, 9, 5) and taken(4, 112, 80, 80, 1, 7, stride=2)
    assert taken(1, 3, 50, 146, 1, 2) and taken(8, 16, 50, 146, 16, 2) and taken(8, 3, 50, 146, 1, 2, stride=2)
