"""The benchmark's printed line is short enough for the tail of a log to hold it whole, and carries the headline unchanged."""
import copy
import json

import bench


def _record():
    fam = {f"gelu[w{n}x128]": dict(bound="mfma", achieved=655.5724727006907, peak=2500.0, unit="TFLOP/s", frac=0.2622289890802762, launches=840 + n,
                                   avg_us=63.74893211094396, total_ms=53.5, traffic=124470000) for n in range(30)}
    fam["draft"] = dict(bound="cu_stream", launches=11, avg_us=140.8, total_ms=1.5, unit="GB/s per CU", achieved_gbs_per_cu=75.1)
    rule = dict(K=2, value=1.5e7 / 7, ms_per_step=44.0 / 7, speedup_vs_target_only=1.0 / 7, acceptance=0.7, mean_committed_per_round=3.0 / 7)
    pred = dict(predicted_rounds=71 / 7, predicted_ms=385 / 7, predicted_speedup_vs_target_only=5 / 7)
    rec = {k: 1.0 / 7 for k in ("target_only_ms", "target_only_steps_per_s", "speedup_vs_target_only", "patch_rate_speedup", "predicted_speedup_eq8",
                                "acceptance", "mean_committed_per_round", "c", "v", "prefill_ms")}
    rec.update(value=25048840.00165835, ms_per_step=58.86739664999965, steps=20, rounds_per_decode=11, resident_launches_per_decode=11, near_ties=2,
               dtype="bf16", workload="cfg3: B=1024", phase_ms=dict(draft=1.4 / 7, verify=7.6 / 7, accept=0.1 / 7, target_step=2.8 / 7),
               planned_block_size={"v_of_K": {str(k): k / 7 for k in range(1, 17)}, "eq8_over_measured_cost_table": rule, "shortest_predicted_batch_decode": rule},
               batch_level_prediction=dict(model="x" * 300, round_ms_by_active={str(k): k / 7 for k in range(20)}, pooled_acceptance=pred, per_series_acceptance=pred),
               roofline=dict(bound="mfma", achieved=655.57, peak=2500.0, unit="TFLOP/s", frac=0.26, traffic=1, kernel="gelu[w128x128]", avg_us=63.7,
                             launches=840, traffic_source="profiles/traffic_cfg3_bench.txt", path="kernel by kernel, " * 6))
    configs = {name: dict(copy.deepcopy(rec), families=fam) for name in bench.ALL_CONFIGS}
    return dict(rec, metric="forecast steps/s", unit="forecast steps/s", n_gpus=1, warmup=5, higher_is_better=True, scaling="weak", vs_baseline=None,
                data="synthetic", config=dict(workload=rec["workload"]), kernel_families=fam, configs=configs)


def test_line_is_short_and_keeps_the_headline():
    out = _record()
    line = bench.compact(copy.deepcopy(out))
    text = json.dumps(line)
    assert len(text) < 9000 < len(json.dumps(out))
    for k in ("metric", "unit", "n_gpus", "steps", "warmup", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert line[k] == out[k]
    for k in ("value", "ms_per_step", "speedup_vs_target_only", "v"):
        assert abs(line[k] - out[k]) <= 1e-5 * abs(out[k])
    assert set(line["configs"]) == set(bench.ALL_CONFIGS)
    assert line["roofline"]["traffic"] == 1 and 0 < len(line["kernel_families"]) <= 8


def test_line_of_an_ablation_run_without_predictions():
    out = _record()
    del out["configs"]
    out.update(planned_block_size=None, batch_level_prediction=None)
    line = bench.compact(out)
    assert line["planned_block_size"] is None and line["batch_level_prediction"] is None
