"""bench.py's command line: this build runs on one GPU only and must say so instead of starting ranks."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode != 0
    assert "ONE GPU" in (r.stdout + r.stderr)
    assert not r.stdout.strip().startswith("{")          # no result line


@pytest.mark.gpu
def test_bench_line_with_lse(gpu_device):
    """With --lse the step itself takes the log-sum-exp; the other legs are timed all the same."""
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--lse", "--no-cpu", "--steps", "4", "--warmup", "1"],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    line = json.loads(r.stdout.strip().splitlines()[-1])
    assert line["config"]["score_mode"] == "lse supplied (one K pass)" and line["value"] > 0
    assert "lse_supplied" not in line and line["ordinary_layer"]["ms_per_step"] > 0
