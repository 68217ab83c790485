"""bench.py times and reports the launches a user gets: without a launch option
the library's own (deep ones, three FP64 steps), with one the shape it names, and
the figures per launch follow the steps that ran.
"""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("options,steps,kernel", [
    (["--workload", "sq256", "--precision", "f32h64"], 5, "deep_kernel"),
    (["--workload", "sq512", "--precision", "f64"], 3, "stepk_kernel"),
    (["--workload", "sq512", "--precision", "f64", "--steps-per-launch", "2"], 2, "stepk_kernel"),
    (["--workload", "sq512", "--precision", "f64", "--block", "256"], 2, "stepk_kernel"),
    (["--workload", "sq512", "--precision", "f64", "--steps-per-launch", "1"], 1, "step_kernel"),
    (["--workload", "sq256", "--precision", "f32h64", "--autotune"], None, None)])
def test_the_line_reports_the_launches_that_ran(require_gpu, tmp_path, options, steps, kernel):
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--steps", "60", "--warmup", "13",
                        "--no-cpu-baseline", *options], capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, TMPDIR=str(tmp_path)))
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads(r.stdout.strip().splitlines()[-1])
    roof, run, cfg = out["roofline"], out["config"]["running"], out["config"]
    k = roof["steps_per_launch"]
    if steps is None:       # the autotuner's choice: either, but what is reported ran
        assert k == run["steps_per_launch"] and (k > 3 or k == cfg["launch"]["steps_per_launch"])
    else:
        assert k == steps == run["steps_per_launch"] and f"lbm::{kernel} " in cfg["step_kernel"]
    assert roof["launch_ms"] == pytest.approx(out["ms_per_step"] * k)
    b = {"f64": 448, "f32h64": 232}[cfg["storage"]]
    assert roof["hbm"]["algorithmic_GBps"] == pytest.approx(b * cfg["nodes"] / (out["ms_per_step"] * k) / 1e6)
