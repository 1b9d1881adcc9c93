"""The rules that keep the kernels' loads inside their buffers, evaluated on the CPU over every small size (no GPU): the same
header functions the kernels and the launchers call; and which shapes they pick for the layers that test those."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "host_rules")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2206_10620_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_rules_main.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules_keep_every_load_in_bounds(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-2000:]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_the_binary32_layers_run_the_shapes_they_are_there_for(program):
    """The dense product's test layers reach the workgroup shapes, and the loop remainders, that they name; every shape is among them."""
    from test_gpu_f32_split import LAYERS
    args = []
    for (n, c_in, c_out, h, w, ks, stride, _), *_ in LAYERS:
        pixels = n * ((h - 1) // stride + 1) * ((w - 1) // stride + 1)
        args += [(c_out + 31) // 32, pixels, ks * ks * ((c_in + 15) // 16), ks * ks * ((c_in + 7) // 8)]
    r = subprocess.run([program] + [str(a) for a in args], capture_output=True, text=True, timeout=120)
    lines = [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    names = {"parts": {row[1] for row in LAYERS}, "whole": {row[3] for row in LAYERS}}
    assert len(lines) == len(LAYERS) + 1
    for (_, parts, share, whole), got in zip(LAYERS, lines):
        assert got == parts + (share,) + whole
    assert lines[-1] == (len(names["parts"]), len(names["whole"]))        # how many shapes there are
