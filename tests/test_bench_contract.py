"""The benchmark's command-line contract: one JSON line with the agreed keys; more than one GPU is refused."""
import json
import subprocess
import sys
from dataclasses import replace
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, str(ROOT / "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def test_columns_per_pass_follow_the_kernel():
    """The four-copy kernels have four columns whatever the number of copies, the padded ones sixteen."""
    from bench import columns_per_pass
    from paper_2501_15129_amd import EsContext
    from paper_2501_15129_amd.workloads import Workload
    base = Workload("paper-base", pop=128, envs=1, horizon=1000, obs=8, hid=256, act=2, dtype=0, noise_dtype=0, seed=5)
    for kw, columns in ((dict(pop=64, episodes=16), 4), (dict(episodes=16), 16), (dict(episodes=8), 4), (dict(dtype=1, noise_dtype=1), 4),
                        (dict(dtype=1, noise_dtype=1, episodes=16), 16), (dict(dtype=1, noise_dtype=1, envs=4, obs=244, act=17), 4),
                        (dict(dtype=1, noise_dtype=1, envs=16, obs=244, act=17), 16), (dict(hid=48, pop=1000, envs=16), 16)):
        kernel = EsContext(replace(base, **kw)).rollout_kernel
        assert "mfma" in kernel and columns_per_pass(kernel) == columns, kw


def test_one_copy_per_workgroup_is_no_matrix_core_kernel():
    """... so that the benchmark prices it against the vector ALU."""
    from paper_2501_15129_amd import EsContext
    from paper_2501_15129_amd.workloads import Workload
    assert "mfma" not in EsContext(Workload("paper-base", pop=128, envs=1, horizon=1000, obs=8, hid=256, act=2, dtype=0, noise_dtype=0, seed=5)).rollout_kernel


@pytest.mark.gpu
def test_bench_prints_one_json_line_with_the_agreed_keys():
    r = subprocess.run([sys.executable, str(ROOT / "bench.py"), "--config", "0", "--steps", "3", "--warmup", "1"],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln for ln in r.stdout.splitlines() if ln.strip()]
    assert len(lines) == 1
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 3 and d["warmup"] == 1 and d["vs_baseline"] is None
    assert d["higher_is_better"] is True and d["data"] == "synthetic" and d["dtype"] == "f32"
    assert "workload" in d["config"] and "model" not in d["config"]
    assert set(("bound", "achieved", "peak", "unit", "frac", "traffic")) <= set(d["roofline"])
    assert d["roofline"]["bound"] in ("hbm", "mfma", "alu")
    assert abs(d["roofline"]["frac"] - d["roofline"]["achieved"] / d["roofline"]["peak"]) < 1e-12
    assert set(("value", "unit", "cores", "kind", "sample")) <= set(d["cpu_baseline"]) and d["cpu_baseline"]["kind"] == "oracle"
    assert d["value"] > 0 and d["ms_per_step"] > 0
