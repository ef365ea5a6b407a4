"""The line that bench.py prints: what it must hold, and its length."""
import json

import pytest

import bench


def _result(calls, words):
    stat = {"us_median": 12345.678, "us_min": 12345.678, "samples": 12, "algorithmic_bytes": 4031999999.0,
            "achieved_GBs": 6619.5, "frac_of_hbm_peak": 0.8274}
    kernels = {f"accumulate_topk_select_{i}": {"kernel": "slot_fill_accumulate_kernel<false, 2>", "us_per_call": stat,
                                               "us_main_kernel": stat} for i in range(calls)}
    batch = {"us_per_launch": 969.8, "frac_of_hbm_peak": 0.255, "plain_gather": {"what": "x" * 200}}
    block = {"workload": "y" * words, "kernels": kernels, "reduce": {"us_per_call": stat}, "reduce_batch": batch}
    return {"metric": "m", "value": 3.3e11, "unit": "elements/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 0.769, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
            "data": "synthetic", "config": {"workload": "z" * 600}, "roofline": {"frac": 0.8},
            "kernels": kernels, "separate_calls_path": {"ms_per_step": 1.0}, "overlapped_path": {"ms_per_step": 1.0},
            "sanity": {"selected_per_iteration": [1, 2, 3]}, "cpu_baseline": {"value": 1.0},
            "per_config": {f"cfg{i}": block for i in range(1, 6)}, "reduce_batch": {f"cfg{i}": batch for i in range(1, 6)}}


@pytest.mark.parametrize("calls,words", [(0, 0), (8, 300), (60, 5000)])
def test_the_line_is_whole_and_short(calls, words):
    out = _result(calls, words)
    text = bench.result_line(out)
    assert "\n" not in text and len(text) <= bench.LINE_MAX
    line = json.loads(text)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config"):
        assert line[key] == out[key]
    if calls <= 8:
        assert set(line["per_config"]) == set(out["per_config"])
        assert line["roofline"] and line["cpu_baseline"]
        assert line["per_config"]["cfg3"]["reduce_batch"]["us"] == 969.8
    else:
        assert "per_config" in line["left_out"]
    for i in range(calls if calls <= 8 else 0):
        assert line["per_config"]["cfg2"][f"accumulate_topk_select_{i}"]["us"] == 12345.678
