"""The span planner on the host, over random launches and devices."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("cus", [8, None, 1024])
def test_span_planner_over_random_launches(tmp_path, cus):
    """tests/c/span_plan.cpp: a span launch's workspace fits what its callers
    are sure to hold, its record places are distinct, and the launch rule and
    the merge's rule draw their lines where they say (256 units by default)."""
    inc = ["-I", os.path.join(ROOT, "tests", "c", "hipstub"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2606_29207_amd", "csrc")]
    exe = tmp_path / "span_plan"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", *inc,
           os.path.join(ROOT, "paper_2606_29207_amd", "csrc", "kf_api.cpp"),
           os.path.join(ROOT, "tests", "c", "span_plan.cpp"), "-o", str(exe), "-lm"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, " ".join(cmd) + "\n" + res.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    run = subprocess.run([str(exe)] + ([str(cus)] if cus else []), capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0 and "span_plan ok" in run.stdout, run.stdout + run.stderr[-4000:]
