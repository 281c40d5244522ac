"""The benchmark's printed line: one JSON object with every field a reader of the
line relies on, within the 2000 characters at the end of the output that are sure
to be kept, however large the full record is."""
import json

import bench


def _record():
    big = {str(i): list(range(50)) for i in range(100)}
    lp = {"live_tflops": 409.88, "deployed_pct_of_optimal_test": 86.56, "speedup_vs_f32_best_time_weighted": 3.497,
          "roofline": big, "chosen": big}
    return {
        "metric": "GEMM TFLOP/s; % of exhaustive-best config; % MFMA peak; selector regret", "value": 130.68,
        "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 164.546, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "w" * 250, "problems": 1200, "gflop_per_step": 21502.765, "k": 8, "selector": "MLP",
                   "chosen": big},
        "pct_mfma_peak": 83.08, "deployed_pct_of_optimal_test": {"geomean": 93.31, "mean": 93.81},
        "pct_of_exhaustive_best": {"time_weighted_live_in_sample": 92.87, "geomean_all_rows_table_in_sample": 94.81},
        "selector_regret_test": {"kmeans_ceiling": 0.0331, "DT-A": 0.0942, "DT-B": 0.0932, "MLP": 0.0653},
        "roofline": {"bound": "mfma", "kernel": "gemm_f32_dma_kernel<128, 128, 8, 32, 0, 1>", "launches_per_step": 44,
                     "achieved": 147.425, "peak": 157.3, "unit": "TFLOP/s", "frac": 0.9372, "traffic": 2202009600,
                     "algorithmic_bytes_per_launch": 590068128, "kernel_ms_per_step": 35.054},
        "cpu_baseline": {"value": 0.0474, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "sample": "s" * 500},
        "lowp": {"bf16": dict(lp), "fp8": dict(lp)}, "vgg16": {"ms_per_inference": {"selector": 0.5686}, "layers": big},
        "grouped_bf16": {"rows_padded_16B": {"ms_per_launch": 0.3689}}, "k_sweep_pct_of_optimal_test": big}


def test_line_is_short_and_whole():
    text = json.dumps(bench.line_of(_record()))
    assert "\n" not in text and len(text) < 2000
    line = json.loads(text)
    for key in bench.CONTRACT + ("config", "roofline", "cpu_baseline"):
        assert key in line
    assert line["value"] == 130.68 and line["vs_baseline"] is None and line["config"]["problems"] == 1200


def test_line_without_the_optional_sections():
    rec = _record()
    for key in ("cpu_baseline", "lowp", "vgg16", "grouped_bf16"):
        del rec[key]
    assert len(json.dumps(bench.line_of(rec))) < 2000
