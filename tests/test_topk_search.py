"""The top-k kernel's search on the host, under the undefined-behaviour sanitizer: right picks, and few
steps whatever the logits' values are.  Midpoints between logits alone need 128 steps from a mask of
the lowest finite value down to ordinary logits; the bound is six steps
that cut outliers off, 16 by value and 32 by key."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_picks_and_steps_of_the_threshold_search(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-o", exe,
                    os.path.join(HERE, "topk_search_driver.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    steps = {line.split(" ", 1)[1]: int(line.split(" ", 1)[0]) for line in r.stdout.splitlines()}
    assert len(steps) == 11 and max(steps.values()) <= 54, steps
    assert max(steps[k] for k in steps if "mask" in k) <= steps["normal"] + 12, steps
