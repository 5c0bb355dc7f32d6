"""Host-side checks of bench.py that need no GPU: the one-GPU rule and the byte accounting."""
import os
import subprocess
import sys

import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in r.stderr and "--gpus 1" in r.stderr
    assert r.stdout.strip() == ""                      # no JSON line that could be mistaken for a measurement


def test_expert_bytes_match_the_shapes():
    sys.path.insert(0, ROOT)
    import bench
    cfg = wl.CONFIGS["mixtral"]
    gu, dn = bench.expert_bytes(cfg, 4)
    assert gu == 4 * 2 * 4096 * 14336 * 2 and dn == 4 * 4096 * 14336 * 2
    cfg = wl.CONFIGS["dsv2lite"]
    gu, dn = bench.expert_bytes(cfg, 10)
    per_expert = 3 * cfg.H * cfg.F * 2
    assert gu + dn == 10 * per_expert + cfg.n_shared * 3 * cfg.H * cfg.F_shared * 2


def test_layer_policy_table():
    sys.path.insert(0, ROOT)
    import pytest

    import bench
    names = bench.layer_policy("0-3:off,4-43:aggressive,44-47:moderate", 48, "aggressive")
    assert names[:4] == ["off"] * 4 and names[4:44] == ["aggressive"] * 40 and names[44:] == ["moderate"] * 4
    assert bench.layer_policy("", 3, "moderate") == ["moderate"] * 3          # layers not named keep the preset
    assert bench.layer_policy("2:off", 4, "moderate") == ["moderate", "moderate", "off", "moderate"]
    for bad in ("0-9:off", "1:sometimes", "3-1:off"):
        with pytest.raises(ValueError):
            bench.layer_policy(bad, 4, "off")


def test_the_line_of_the_full_report_is_short():
    """What goes to stdout keeps the agreed fields and stays below 4000 characters however many settings were measured."""
    import json
    sys.path.insert(0, ROOT)
    import bench
    agreed = dict(metric="MoE-stack decode us/batch (48 chained layers)", value=4000.1, unit="us/batch", n_gpus=1, steps=20,
                  warmup=5, ms_per_step=4.0001, higher_is_better=False, scaling="weak", vs_baseline=None, dtype="bf16",
                  data="synthetic", config={"workload": "w" * 600}, roofline={"kernel": "k" * 600}, cpu_baseline={"sample": "s" * 400})
    entry = dict(us_graph_wall=12345.6, detail="d" * 400)
    report = dict(agreed, stack={f"T{t}_{p}": entry for t in (32, 128, 256, 512) for p in bench.PRESET_NAMES},
                  configs=[dict(us=100.0, detail="d" * 400)] * 45, mixtral_T8=dict(value=120.5, detail="d" * 2000))
    line = bench.headline_line(report)
    assert all(line[k] == v for k, v in agreed.items())
    assert line["stack_us"]["T512_aggressive"] == 12345.6 and line["mixtral_T8_us"] == 120.5
    assert len(json.dumps(line)) < 4000
