"""The benchmark's result line: one line of JSON on the standard output that
holds the contract's keys and stays short enough to be taken whole from a log
(16 kB were cut); the full record goes to the standard error output."""
import json
import types

import bench

KEYS = {"metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better",
        "scaling", "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"}


def _stat(v):
    return {"median": v, "p10": v / 3, "p90": v / 0.7, "mean_iqr": v / 0.9, "n": 10000}


def _record():
    """As many measurements as the benchmark makes, all digits long."""
    lat = {"empty_e2e_us": _stat(92.0 / 9.7), "ratio_to_empty_median": 1.0 / 0.9,
           "cache_stats": {"calls": 24202}, "host_cost_ns": {"scan": {"1": 2.5 / 0.9}}}
    lat.update({f"decode_chain_number_{i}_e2e_us": _stat(10.0 / (i + 3)) for i in range(24)})
    for n in ("mixed_stream", "mixed_stream_autotuned", "mixed_stream_generic",
              "mixed_stream_resident"):
        lat[n] = {"calls": 10000, "tuning": {"kept": {str(i): [[0, 1]] for i in range(9)}},
                  "hit_e2e_us_by_tokens": {str(i): _stat(10.0 / (i + 3)) for i in range(9)}}
    bw = {f"op_{i}_rows65536": {"bytes": 1 << 30, "mean_us": 81.0 / 0.7, "GB/s": 6e3 / 0.7,
                                "frac_of_peak": 0.8 / 0.7, "matched_ceiling": "1 read : 1 write",
                                "frac_of_matched_ceiling": 0.9 / 0.7} for i in range(24)}
    bw["copy_ceiling_GB/s"] = 6400.0 / 0.7
    return lat, bw


def test_result_line(capsys):
    args = types.SimpleNamespace(steps=20, warmup=5)
    lat, bw = _record()
    for bandwidth in (bw, None):
        bench.emit(args, _stat(10.4), 0.0002, lat, bandwidth, {"frac": 0.8}, {"value": 1528.0})
        out, err = capsys.readouterr()
        assert out.endswith("\n") and out.count("\n") == 1 and len(out) < 8000
        line, full = json.loads(out), json.loads(err)
        assert KEYS <= set(line) and line["value"] == 10.4 and line["steps"] == 20
        assert line["latency"]["empty_e2e_us"] == 9.4845
        assert line["latency"]["mixed_stream"]["hit_e2e_us_by_tokens"]["8"] == 0.90909
        assert full["latency"] == json.loads(json.dumps(lat)) and full["bandwidth_8192"] == bandwidth
    assert line["bandwidth_8192"] is None
    assert bench.brief({"median": 2.0 / 3}) == 0.66667
