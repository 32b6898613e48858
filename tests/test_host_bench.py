"""The line bench.py prints: one line of JSON, short, with the headline first and the layer tables in a file."""
import json

import bench


def test_the_line_is_short_and_whole(tmp_path):
    one = dict(ms=0.1234567891, kernel="mfma_p4_bf16_lut", flops_algorithmic=155222802432.0, flops_executed=155222802432.0,
               conv_equivalents_paper=4, conv_equivalents_executed=1.0, bytes_algorithmic=235028480, tflops_paper_count=1209.62,
               tflops_executed=316.36, bound="mfma", roof_ms=0.0329, frac_of_roof=0.1265)
    passes = {n: dict(one) for n in bench.PASSES}
    layer = dict(workload="C3: N=4 Cin=128 Cout=128 128x128 R=16 bilinear G=16, fused fwd+bwd_data+bwd_weight", dtype="f32",
                 ms_per_step=0.71234567, frac_of_roof=0.25, passes=passes)
    step = dict(workload="C5: " + "x" * 150, ms_per_step=28.4123456789, rotconv_frac_of_roof=0.41,
                ms_by_call={f"rotconv_call_{i}": 1.2345 for i in range(14)},
                layers={f"enc{i}a": dict(shape="512->512 @64x64 R=16", passes=passes) for i in range(18)})
    out = dict(metric="rotconv_fwd_bwd_tflops", value=134.6683455144003, unit="TFLOP/s", n_gpus=1, steps=20, warmup=3,
               ms_per_step=0.8880185999998957, config=dict(workload="C2", passes=passes),
               c3_r16_layer=dict(f32=layer, bf16=layer), c2_r4_layer_bf16=layer,
               unet_train_step=dict(C4=step, C5=step, C5_bf16=step))
    before = json.dumps(out)
    text = bench.the_line(out, str(tmp_path / "layers.json"))
    assert "\n" not in text and len(text) < 7000
    line = json.loads(text)
    assert [line[k] for k in ("metric", "value", "ms_per_step")] == [out[k] for k in ("metric", "value", "ms_per_step")]
    assert line["config"]["passes"]["rotconv_pool_fwd"]["flops_executed"] == one["flops_executed"]
    assert line["unet_train_step"]["C5"]["ms_by_call"] == step["ms_by_call"]
    assert json.dumps(out) == before and json.load(open(tmp_path / "layers.json")) == json.loads(before)
