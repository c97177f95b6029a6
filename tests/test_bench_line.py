"""The line that bench.py prints is read from the end of a run's output: it has to fit there, whole, with every field of its
contract."""
import argparse
import json

import bench

LIMIT = 5000


def fake_result(c):
    x = 0.123456789012345678 * (c + 1)
    kernels = {"gather": x, "priority_pass": x, "deferred_pass": x}
    r = {k: x * 1e9 for k in bench.PER_CONFIG}
    r.update(workload=f"configs[{c}] a_name: " + "8 tables per shard, rows and dims of each, IDs, batches cycled " * 5, dtype="f32",
             ms_per_step=x, kernel_avg_us=kernels, schedule="s" * 300, ids_per_batch=[[297014] * 10] * 8,
             host_phase_us_per_step_and_group=[kernels] * 8, step_without_index_chains={"us_per_step": x, "note": "n" * 300},
             roofline={"bound": "hbm", "kernel": "class_pass_kernel", "achieved": x, "peak": 8000.0, "unit": "GB/s", "frac": x,
                       "traffic": x, "note": "n" * 400, "all_kernels": {k: kernels for k in "abc"}},
             cpu_baseline={"value": x, "unit": "rows/s", "cores": 1, "kind": "oracle", "ms_per_step": x, "sample": "s" * 400},
             isolated_kernels={str(i): kernels for i in range(12)}, load_balancer_path={str(i): kernels for i in range(12)})
    return r


def test_the_line_is_short_and_whole():
    args = argparse.Namespace(steps=50, warmup=10, blocks=10)
    configs = [2, 1, 3, 4]
    results = {c: fake_result(c) for c in configs}
    assert len(json.dumps(results)) > 8192                   # what used to be printed
    text = json.dumps(bench.result_line(args, configs, results, {"name": "gpu" * 10, "memory_GiB": 287.98765432101}))
    assert len(text) < LIMIT and "\n" not in text
    line = json.loads(text)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config", "roofline", "cpu_baseline", "per_config"):
        assert k in line, k
    assert (line["n_gpus"], line["steps"], line["warmup"], line["dtype"], line["data"]) == (1, 50, 10, "f32", "synthetic")
    assert abs(line["value"] / results[2]["value"] - 1) < 1e-5 and abs(line["ms_per_step"] / results[2]["ms_per_step"] - 1) < 1e-5
    assert sorted(line["per_config"]) == ["configs[1]", "configs[2]", "configs[3]", "configs[4]"]
