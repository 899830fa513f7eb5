"""Host-only check (no GPU) of the geometry of the line grids: with every number
of line classes, radius, span and number of grains there is a grid, and its
cells list what the lines that look at them need."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1311_5334_amd", "csrc")


def test_line_grids(tmp_path):
    exe = str(tmp_path / "line_grid_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", "/opt/rocm/include", "-I" + CSRC,
                           os.path.join(HERE, "native", "line_grid_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "line grid ok" in r.stdout
