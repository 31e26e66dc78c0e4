"""The bench's JSON line (no GPU needed): whole within what is kept of its output, the headline's fields in it untouched."""
import json

import bench


def _record(i):
    return {"workload": "S16_bf16_kn_%02d" % i, "note": "a streaming product " * 3, "dtype": "bf16", "M": 16, "N": 28672, "K": 8192,
            "plan": "variant=%d:bf16_skinny_m16n256k64s4_nn tile=16x256x64 threads=512 stages=4 lds=139264 split=2 ktiles/slice=64 "
                    "grid=224 (tiles 1x112) group_m=1 workspace=3670016 unaligned=bf16_r64x64_nn streamk=0 rot=0,0 pack=0 acopy=0" % i,
            "ms_per_step": 0.08172574499994312, "event_ms_per_step": 0.08156742095947266, "tflops": 91.968482734605,
            "tflops_events": 92.14699544974546, "gbs_events": 5773.649460291146, "torch_tflops": 71.1234567891, "pct_of_library": 129.3081,
            "per_launch_ms": {"median": 0.08335000276565552, "min": 0.08138900250196457, "mean": 0.0837, "launches": 200},
            "roofline": {"bound": "hbm", "achieved": 5773.649460291146, "peak": 8000.0, "unit": "GB/s", "frac": 0.7217061825363933, "traffic": None},
            "cpu_baseline": {"value": 0.011688400123591526, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "sample": "some rows " * 10}}


def _headline():
    return {"metric": "GEMM TFLOP/s", "value": 1538.4246924108665, "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 0.7146903350000384, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
            "data": "synthetic", "config": {"workload": "C3 " * 30, "plan": _record(0)["plan"]}, "roofline": _record(0)["roofline"],
            "pct_of_peak": 61.1, "per_launch_ms": _record(0)["per_launch_ms"], "rocm_smi": {"before": "x" * 100, "after": "x" * 100}}


def test_line_of_a_full_run_is_short_and_complete():
    out, records = _headline(), [_record(i) for i in range(21)]
    line = bench.result_line(out, records)
    assert len(line) <= bench.LINE_LIMIT and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config"):
        assert got[k] == out[k], k
    assert [w["name"] for w in got["workloads"]] == [r["workload"] for r in records]
    for w, r in zip(got["workloads"], records):
        assert abs(w["tflops"] - r["tflops"]) <= 1e-3 * r["tflops"] and w["plan"] == "bf16_skinny_m16n256k64s4_nn/2"
    assert out == _headline()                                          # (the caller's record is left as it was)


def test_line_that_would_be_too_long_keeps_the_contract_fields():
    out = dict(_headline(), rocm_smi={"before": "x" * 9000})
    got = json.loads(bench.result_line(out, [_record(0)]))
    assert "rocm_smi" not in got and got["value"] == out["value"] and len(got["workloads"]) == 1
