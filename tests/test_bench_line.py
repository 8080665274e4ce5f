"""The line that bench.py prints: one JSON object, small enough to be recorded whole."""
import json

import bench


def test_the_line_is_whole_and_small():
    x = 68.12345678901234
    nested = {f"key_{i}": {"us": x * i, "algorithmic_bytes": 402653184, "hbm_gbps": x * 77.7} for i in range(20)}
    result = {"metric": "loki_decode_attn_us_per_step", "value": x, "ms_per_step": x / 1e3, "steps": 20, "dtype": "bf16",
              "vs_baseline": None, "kernels_us": {"fused_decode": x}, "nested": nested}
    entries = [{**{c: x for c in bench.CONFIG_COLUMNS}, "workload": "large_share", "B": 64, "select_mode": i % 2, "frac_of_peak": None,
                "kernels_us": {"rotate_score": x, "select_attend": x}} for i in range(26)]
    text = bench.result_line(result, entries)
    line = json.loads(text)
    assert "\n" not in text and len(text) < 8000
    assert line["value"] == x and line["ms_per_step"] == x / 1e3  # the measured value in full
    assert line["nested"]["key_3"]["us"] == float(f"{3 * x:.5g}") and line["nested"]["key_3"]["algorithmic_bytes"] == 402653184
    assert line["configs"]["columns"] == list(bench.CONFIG_COLUMNS) and len(line["configs"]["rows"]) == 26
    assert line["configs"]["rows"][1][:2] == ["large_share", 64] and line["configs"]["rows"][1][7] == 1
    assert json.loads(bench.result_line(result, None))["configs"] is None
