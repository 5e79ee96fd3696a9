"""The JSON line bench.py prints on stdout (no GPU): every field a reader needs, in fewer than 8000 characters."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench


def test_the_line_on_stdout_is_short_and_keeps_the_figures():
    phases = {"unit": "u", "phases": [{"phase": "x" * 80, "at_us": 1.23, "us": 0.12, "mflop": 0.4, "pct_of_team_fp32_peak": 1.2}] * 20}
    row = {"name": "paper-cifar-100maps", "arch": "3x32x32-100C3", "mode": "resident", "kernels": "k" * 130, "bound": "fp32",
           "train": {"images_per_s": 12345.6, "us_per_image": 81.0, "images": 4000}, "frac": 0.02345,
           "forward_only": {"images_per_s": 23456.7, "us_per_image": 42.0}, "achieved_tflops": 1.2345, "achieved_gbs": 123.45,
           "traffic": 10324187078, "per_layer": phases, "dependency_bound": {"kind": "k" * 150, "us": 4.1},
           "cpu_baseline": {"value": 1234.5, "unit": "images/s", "sample": "s" * 100}, "paper_context": "p" * 190}
    out = {"metric": "online-training images/sec", "value": 63794.6, "unit": "images/s", "n_gpus": 1, "steps": 60, "warmup": 5,
           "ms_per_step": 15.6753, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
           "data": "synthetic", "config": {"workload": "w" * 200}, "roofline": {"bound": "hbm", "frac": 0.01, "per_layer": phases,
           "dependency_bound": {"kind": "k" * 150}}, "per_config": [row] * 12, "extra": {"e%02d" % i: 1234567.8 for i in range(40)},
           "cpu_baseline": {"value": 2167.2, "sample": "s" * 120}}
    line = json.dumps(bench.short(out))
    assert len(line) < 8000
    got = json.loads(line)
    assert set(got) == set(out) and all(got[k] == out[k] for k in out if k not in ("roofline", "per_config"))
    assert got["roofline"]["frac"] == 0.01
    assert got["per_config"][3]["train_images_per_s"] == 12345.6 and got["per_config"][3]["cpu_images_per_s"] == 1234.5
    assert "per_layer" in out["roofline"] and "per_layer" in out["per_config"][0]   # (what stderr gets is whole)
