"""The benchmark's result line: every key of the contract, and short enough to survive in the last 8000 characters
of the output, whatever the number of calls that were timed."""
import json

import bench

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config", "roofline")


def _result():
    out = {k: "x" * 60 for k in CONTRACT}
    out["config"], out["roofline"], out["cpu_baseline"] = {"workload": "x" * 1000}, {"kernel": "x" * 1000}, {"sample": "x" * 600}
    call = {"layer": "fc1", "call": "bwd_input", "path": "dense-mfma", "avg_ms": 0.123456, "note": "x" * 150}
    slowest = {"call": "fc1/bwd", "avg_ms": 0.123456, "bound": "mfma", "frac": 0.1234, "hbm_frac": 0.1, "alu_frac": 0.2, "lds_frac": None}
    out["calls"] = [call] * 100
    out["sweep"] = [dict(position=k, density=0.1, next_density=0.02, steps=4, ms_per_step_device=3.1234, eff_tflops=123.456,
                         path="dense-mfma", nnz={"fc1": 6553600}) for k in range(6)]
    out["per_config"] = [dict(config="C%d" % k, workload="x" * 260, dtype="bf16-in/f32-acc", ms_per_step=1.2345, eff_tflops=12.3456,
                              hbm_frac=0.1234, alu_frac=0.1234, ms_per_mask_update=0.1234, slowest_call=slowest, calls=[call] * 12,
                              graph_replay={"ms_per_step": 1.1, "replays": 50, "matches_call_by_call": True, "holds": "x" * 90},
                              dense_grad_gemm={"layers": "x" * 700}, sparse_pinned={"ms_per_step": 1.3, "calls": [call] * 12})
                         for k in range(1, 5)]
    return out


def test_result_line_is_short_and_whole(capsys, tmp_path):
    out = _result()
    bench.emit(out, str(tmp_path / "full.json"))
    bench.emit(out, None)
    got = capsys.readouterr()
    lines = got.out.splitlines()
    assert len(lines) == 2 and lines[0] == lines[1] and len(lines[0]) < 7500
    line = json.loads(lines[0])
    assert all(line[k] == out[k] for k in CONTRACT)
    assert [row["config"] for row in line["per_config"]] == ["C1", "C2", "C3", "C4"] and len(line["sweep"]) == 6
    assert json.loads(got.err) == out == json.loads((tmp_path / "full.json").read_text())
