"""bench.py's line on stdout: the keys its readers need, and a length that the tail of a log holds whole."""
import json

import bench


def test_short_line_is_short_and_complete():
    layer = dict(name="x" * 20, note="n" * 500, **{"f%d" % i: 1234.5678 for i in range(16)})
    out = dict(metric="m" * 120, value=1.0, unit="TOPS", n_gpus=1, steps=20, warmup=5, ms_per_step=1.0, higher_is_better=True,
               scaling="weak", vs_baseline=None, dtype="int8", data="synthetic", config=dict(workload="w" * 90, layers=24),
               frac_int8_peak=0.2, event_overhead_us_per_launch=2.4, roofline=dict(layer, traffic_source="t" * 300),
               quant_act_roofline=dict(layer, traffic_source="t" * 300), target_layer=layer,
               cpu_baseline=dict(value=0.08, sample="s" * 150, one_thread=dict(layer)), layers=[layer] * 24, vendor_int8_gemm=dict(rows=[layer] * 3),
               configs=[dict(config=c, layers=30, ms_per_step=1.0, value=2.0, unit="TOPS", shapes=[layer] * 6) for c in (1, 3, 4, 5)])
    line = bench.short_line(out)
    assert len(json.dumps(line)) < 3500
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
              "data", "config", "roofline", "quant_act_roofline", "cpu_baseline"):
        assert k in line
    assert [c["value"] for c in line["configs"]] == [2.0] * 4 and "layers" not in line
