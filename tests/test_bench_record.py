"""What bench.py reports beside its timings, without a GPU."""

import json

import bench
import paper_2510_16045_amd as ams


def test_traffic_is_reported_for_the_kernel_that_was_profiled_only():
    column = bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "column_kernel")
    assert column == 79206371 + 57344
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "multi_kernel") is None
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "slice_kernel") == 79165645 + 57344
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 2, "column_kernel") is None


def test_printed_record_fits_where_8000_characters_are_kept():
    # a whole default run: 8 layer rows, 24 of the batch sweep, 18 of the 70B set, 4 of the vocabulary projection, 24 of the
    # MLP-down shapes, every number with as many digits as a measurement has
    def row(layer, M, fmt):
        num = {k: 123.456789 for k in (
            "us", "us_static_ws", "us_cache_resident", "bare_read_us", "frac_of_bare_read", "GBps", "hbm_frac", "fp16_us", "fp16_ws_us",
            "library_gemm_fp16_us", "speedup_vs_fp16", "speedup_vs_best_fp16", "speedup_static_ws_vs_best_fp16", "best_speedup_vs_best_fp16")}
        return {"layer": layer, "N": 128256, "K": 28672, "M": M, "fmt": fmt, "us_percentiles": {"p10": 123.456}, "us_group_scales": None, **num}

    fmts = ("fp5.33-e2m3", "fp4.25-e2m2")
    table = lambda names, Ms: [row(n, M, f) for n in names for M in Ms for f in fmts]
    line = {
        "metric": "packed_weight_GBps", "value": 3487.2, "unit": "GB/s", "n_gpus": 1, "steps": 200, "warmup": 20, "ms_per_step": 0.07494,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f16", "data": "synthetic", "config": {"workload": "w" * 560},
        "roofline": {"kernel": "k" * 160, "frac": 0.6789}, "single_linear_4096x4096_fp533_m1": {"us": 5.321}, "paper_context": "p" * 112,
        "cpu_baseline": {"value": 0.04227411667899894, "kind": "oracle", "sample": "s" * 290, "per_layer": [{"layer": "qkv", "ms": 282.2}] * 8, "full_configs": {}},
        "layers": table(("qkv", "o", "gate_up", "down"), (1,)), "batch_sweep": table(("gate_up", "down"), (1, 2, 4, 8, 16, 32)),
        "llama70b": table(("o", "gate_up", "down"), (1, 4, 8)), "lm_head": table(("lm_head",), (1, 8)),
        "qwen_down": table(("qwen3-4b", "qwen2.5-7b", "qwen3-32b"), (1, 4, 16, 32)),
    }
    text = json.dumps(bench.printed_record(line), separators=(",", ":"))
    assert len(text) < 7800
    back = json.loads(text)
    assert {k: back[k] for k in ("metric", "value", "unit", "ms_per_step", "config", "roofline")} == {k: line[k] for k in ("metric", "value", "unit", "ms_per_step", "config", "roofline")}
    assert len(back["batch_sweep"]) == 24 and len(back["qwen_down"]["rows"]) == 24 and len(back["llama70b"]["rows"]) == 18
    none = dict(line, batch_sweep=None, llama70b=None, lm_head=None, qwen_down=None, cpu_baseline=None)
    assert all(bench.printed_record(none)[k] is None for k in ("batch_sweep", "llama70b", "lm_head", "qwen_down", "cpu_baseline"))


def test_the_kernel_of_a_launch_is_the_one_its_plan_starts_with():
    from types import SimpleNamespace

    for N, K, M, kernel in ((28672, 4096, 1, "slice_kernel"), (11003, 4099, 5, "slice_kernel"), (28672, 4099, 5, "column_kernel"), (57344, 8192, 1, "multi_kernel")):
        assert bench.dominant_kernel(ams, SimpleNamespace(N=N, K=K), "fp5.33-e2m3", M) == kernel
