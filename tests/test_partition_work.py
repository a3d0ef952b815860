"""What the annealer spends on the binary32 sums that it tries first is worth it: never more than a few trial sums beyond the
binary64 sums alone, on few tokens, on ties and on many tokens, with the same result."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_binary32_sums_cost_no_more_than_they_save(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wno-psabi", "-x", "c++", os.path.join(HERE, "partition_work_driver.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    lines = r.stdout.splitlines()
    assert r.returncode == 0, "\n".join(line for line in lines if ": ok" not in line)
    assert len(lines) == 12 * 4 * 3 * 6 + 18
