"""bench.py's result line: parses, holds the headline and the times of every execution and configuration, and is short
enough to be whole at the end of a log of which 2000 characters are kept."""
import json

import bench

V = 123456.78901234567


def record():
    r = {"kernel": "svdq_linear_w4a4_e3m2 (gemm_e3m2_kernel), 6 launches per step", "bound": "mfma", "achieved": V, "peak": 10100.0,
         "unit": "TFLOP/s", "frac": V, "traffic": 55069955074, "algorithmic_ops": V * 1e9, "clock_ghz_under_this_kernel": V,
         "avg_ms": V, "min_ms": V, "frac_of_int8_peak": V, "traffic_unit": "bytes per step (6 launches)"}
    ex = {"what": "x" * 200, "value": V, "unit": "TOPS", "ms_per_step": V, "roofline": r, "roofline_quantize": r, "per_shape": [r] * 3,
          "weight_bytes_resident": 10 ** 9, "weight_staging_bytes": 10 ** 8, "act_bytes_per_token": {"5120": V, "13824": V},
          "weight_expand_ms_per_step": V}
    names = ("e3m2_prepacked", "int4", "mxfp4")
    return {"metric": bench.METRIC, "value": V, "unit": "TOPS", "n_gpus": 1, "steps": 40, "warmup": 5, "ms_per_step": V,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "x" * 125, "data": "synthetic",
            "config": {"workload": "x" * 260, "execution": "e3m2", "step": "x" * 120, "settle_launches": 40}, **ex,
            "int8_mfma_kernel_pct_of_int8_peak": V, "pct_of_int8_peak_equivalent": V, "context": {"note": "x" * 100},
            "executions": {n: ex for n in names}, "cpu_baseline": {"value": V, "unit": "TOPS", "cores": 16, "kind": "oracle",
                                                                   "sample": "x" * 200, "quantize_GBs": V, "seconds": V},
            "configs": {c: {"workload": "x" * 100, "e3m2": ex, **{n: ex for n in names}} for c in ("c2_attn_o", "c3_ffn_up", "c4_ffn_down")}}


def test_result_line_is_whole_and_short():
    line = bench.result_line(record())
    assert len(line) < 1950 and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
              "data", "config", "roofline", "roofline_quantize", "cpu_baseline"):
        assert k in got, k
    assert got["value"] == 123457.0 and got["roofline"]["frac"] == 123457.0 and got["steps"] == 40
    assert set(got["executions_ms"]) == {"e3m2_prepacked", "int4", "mxfp4"}
    assert set(got["configs_ms"]["c4_ffn_down"]) == {"e3m2", "e3m2_prepacked", "int4", "mxfp4"}
