"""bench.py's printed line: the keys its readers rely on, within a size that survives being cut to the last kilobytes."""
import json

import bench


def _record():
    third = 1.0 / 3.0
    roof = {"bound": "hbm", "kernel": "some_kernel_with_a_long_name_mfma_wide", "achieved": 1000 * third, "peak": 8000.0, "unit": "GB/s", "frac": third,
            "traffic": 123456789.0 * third, "algorithmic_bytes": 1e9 * third, "kernel_ms": third}
    stats = {"median": third, "std": third, "min": third, "max": third}
    kernels = {f"kernel_number_{n}_of_the_schedule": third for n in range(6)}
    cpu = {"value": third, "unit": "GFLOP/s", "cores": 16, "kind": "oracle", "sample": "first 50000000 of 50000000 nonzeros " * 4,
           "seconds": third, "runs_s": [third] * 3}
    sched = {"ms_per_step": third, "ms_per_step_stats": stats, "schedule_flops": third, "gflops": third, "kernels_ms": kernels, "workspace_bytes": 1 << 30,
             "chosen": ["fused", 2], "roofline": roof}
    per = [dict(config_id=n, workload=bench.WORKLOAD_TEXT[n], dtype="f32", nnz=50_000_000, tiles=90_000, steps=20, ms_per_step=third,
                ms_per_step_stats=stats, schedule_flops=third, gflops=third, algorithmic_gbs_whole_step=third, roofline=roof, mfma_busy=third,
                kernels_ms=kernels, setup_s={"generate": third}, fused_vs_fissioned_speedup=third, fused_vs_linear_speedup=third, cpu_baseline=cpu,
                fissioned={"ms_per_step": third, "kernels_ms": kernels, "traversal": dict(kernel="t", ms=third, gbs=third, frac=third)},
                linear={"ms_per_step": third, "gflops": third}) for n in (1, 2, 3, 4, 5)]
    five = {k: sched for k in ("schedule2_fused", "schedule2_fissioned", "schedule1", "schedule3", "linear")}
    nxt = {n: {"workload": "all-mode TTMC, motivating case " * 5, "schedules": five, "cpu_baseline": cpu} for n in "abcde"}
    nxt["ttmc_all_rank_sweep"] = [{"L": 128, "M": 128, "N": 128, "ms": third, "mean_ms": third, "evaluator": "candidate " * 20}] * 11
    head = dict(metric="effective GFLOP/s of the fused schedule (schedule flops / step time) per contraction, 1 MI355X", value=10000 * third, unit="GFLOP/s",
                n_gpus=1, steps=20, warmup=5, ms_per_step=third, ms_per_step_stats=stats, higher_is_better=True, scaling="weak", vs_baseline=None,
                dtype="f32", data="synthetic", config={"workload": bench.WORKLOAD_TEXT[5], "schedule": "fused"}, roofline=roof, schedule_flops=third,
                paper_context=bench.PAPER_CONTEXT, cpu_baseline=cpu, kernels_ms=kernels, fissioned=per[0]["fissioned"], linear=per[0]["linear"])
    return dict(head, per_config=per, next_workloads=nxt)


def test_line_is_short_and_whole():
    rec = _record()
    line = bench.result_line(rec)
    assert "\n" not in line and len(line) < 8000, len(line)
    got = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config",
                "roofline", "cpu_baseline"):
        assert key in got, key
    assert abs(got["value"] - rec["value"]) <= 1e-5 * rec["value"]
    assert [c["config_id"] for c in got["per_config"]] == [1, 2, 3, 4, 5]
    assert all(c["roofline"]["kernel_ms"] and c["linear_ms"] and c["fissioned"]["ms_per_step"] for c in got["per_config"])
    assert len(got["next_workloads"]["ttmc_all_rank_sweep"]) == 11 and len(got["next_workloads"]["a"]["schedules"]) == 5


def test_line_of_a_single_workload():
    """Without the optional schedules and further workloads."""
    rec = _record()
    del rec["next_workloads"], rec["cpu_baseline"]
    rec["per_config"] = [{k: v for k, v in rec["per_config"][0].items() if k not in ("fissioned", "linear", "cpu_baseline", "mfma_busy")}]
    got = json.loads(bench.result_line(rec))
    assert len(got["per_config"]) == 1 and "next_workloads" not in got
