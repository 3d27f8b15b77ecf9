"""The geometry that host and kernels share, run on the CPU."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_pairs_cover_every_row_once(tmp_path):
    exe = str(tmp_path / "route_geometry")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-o", exe, os.path.join(HERE, "models", "route_geometry.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout
