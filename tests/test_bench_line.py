"""The line bench.py prints: every contract field as measured, the legs' main numbers, and short enough to be captured whole."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

CONTRACT = ["metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
            "dtype", "data", "config"]


def record():
    """A record of the shape main() builds, every leg with more in it than the line has room for."""
    many = {f"detail{i}": {"mean_ms": 1 / 3, "samples": [1 / 7] * 20} for i in range(40)}
    leg = lambda **kw: {"note": "x" * 400, **kw, **many}
    roof = lambda **kw: leg(kernel="k_some (all of it)", bound="hbm", achieved=1000 / 3, peak=8000.0, unit="GB/s", frac=1 / 3, ms_call=1 / 3, traffic=None, **kw)
    return {"metric": "m", "value": 3645476825543.1025, "unit": "u", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 11.01554714999935,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u64", "data": "synthetic",
            "config": {"workload": "w", "lanes": 4}, "pipeline": {m: leg(serial_ms=13.7 / 3, four_lanes_ms=11 / 3) for m in ("a", "b", "c")},
            "per_kind": many, "configs": [leg(config=i, name=f"n{i}", folded_prepared_calls=leg(ms_beaver_calls=1 / 3, call_frac_of_int8_peak=1 / 7)) for i in range(5)],
            "config1_step": leg(ms_step=0.6 / 7, workload="w" * 200), "value_definition": {"value": "v" * 300},
            "roofline": roof(kernel_only=leg(achieved=1 / 3, frac=1 / 9, ms=1 / 5)), "roofline_relu": roof(copy_exchange=leg(ms_call=1.2, frac=0.7, traffic=None)),
            "roofline_relu_msb": roof(), "three_party": leg(ms_relu_call=2.4), "cpu_baseline": leg(value=1.25e10, cores=16)}


def test_line_is_short_and_keeps_the_contract():
    import bench
    out = record()
    line = json.dumps(bench.brief(out))
    assert "\n" not in line and len(line) < 6000
    got = json.loads(line)
    for k in CONTRACT:
        assert got[k] == out[k], k                       # whole, not rounded
    assert got["pipeline"]["a"] == {"serial_ms": 4.5667, "four_lanes_ms": 3.6667}
    assert got["configs"][4] == {"name": "n4", "ms_beaver_calls": 0.33333, "call_frac_of_int8_peak": 0.14286}
    assert got["roofline"]["kernel"] == "k_some" and got["roofline"]["frac"] == 0.33333 and got["roofline"]["traffic"] is None
    assert got["roofline_relu"]["copy_exchange"] == {"ms_call": 1.2, "frac": 0.7, "traffic": None}
    assert got["cpu_baseline"] == {"value": 1.25e10, "cores": 16}


def test_line_without_the_optional_legs():
    import bench
    out = record()
    for k in ("configs", "three_party", "cpu_baseline"):
        del out[k]
    got = bench.brief(out)
    assert not {"configs", "three_party", "cpu_baseline"} & set(got) and got["value"] == out["value"]
