"""How the workgroups of the small-tile kernels share their tiles, on the host, under the undefined-behaviour
sanitizer: every tile once, and groups of a row or two spread over all workgroups."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_tile_once_and_even_shares(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-o", exe,
                    os.path.join(HERE, "row_blocks_driver.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
