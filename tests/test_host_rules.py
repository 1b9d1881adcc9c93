"""The rules that keep the kernels' loads inside their buffers, evaluated on the CPU over every small size (no GPU): the same
header functions the kernels and the launchers call."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules_keep_every_load_in_bounds(tmp_path):
    exe = str(tmp_path / "host_rules")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2206_10620_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_rules_main.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-2000:]
