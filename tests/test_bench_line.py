"""The benchmark's result line: one short line with the headline, whatever else was measured."""
import json

import bench


def test_result_line_is_short_and_whole():
    roof = {k: 5555.555555555555 for k in ("achieved", "peak", "frac", "traffic", "traffic_gbs",
                                           "avg_launch_us", "bytes_per_update", "floor_us",
                                           "floor_gbs", "frac_of_floor", "updates_per_launch")}
    out = {"metric": bench.METRIC, "value": 4.6e10, "unit": "link updates/s", "n_gpus": 1,
           "steps": 500, "warmup": 20, "ms_per_step": 0.46123456789012345,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
           "data": "synthetic", "config": {"workload": "x" * 200, "dims": [48] * 4, "beta": 6.0,
                                           "links": 4 * 48 ** 4, "mode": "plain KP"},
           "roofline": {**roof, "bound": "hbm", "unit": "GB/s", "traffic_unit": "y" * 100,
                        "kernel": "pass_kernel"},
           "plaquette_mean_last_half": 0.87, "timed_sweeps": {"z": list(range(1000))},
           "autotuned_us_per_sweep": 463.4,
           "launch": {"block": 256, "flags": 257, "tile_z": 8, "tile_t": 8, "grid_cap": 0},
           "other_configs": {"w": list(range(5000))},
           "learned_vs_plain": {
               "plain": {"link_updates_per_s": 4.7739291066e10, "q": list(range(500))},
               "learned": {"link_updates_per_s": 4.2722684552e10},
               "learned_over_plain_effective": 0.8530326167910421,
               "learned_overrelaxed_over_plain_overrelaxed_effective": 1.8958514141859937},
           "cpu_baseline": {"value": 1.5e7, "unit": "link updates/s", "cores": 16, "kind": "oracle",
                            "sample": "s" * 300, "host": {"model": "m"}}}
    line = json.dumps(bench.result_line(out))
    assert len(line) < 1800 and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
              "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert got[k] == out[k]
    assert got["roofline"]["frac"] == roof["frac"]
    del out["cpu_baseline"], out["learned_vs_plain"]
    assert not {"cpu_baseline", "learned_vs_plain"} & set(bench.result_line(out))
