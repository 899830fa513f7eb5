"""Host-only check (no GPU) of the seed pass's row numbering: a row of a box of
cells is of the layer that an integer division gives, up to the most cells a
view can have (cells of one unit across, given by the caller)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1311_5334_amd", "csrc")


def test_layers_of_rows(tmp_path):
    exe = str(tmp_path / "seed_rows_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", "/opt/rocm/include", "-I" + CSRC,
                           os.path.join(HERE, "native", "seed_rows_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "seed rows ok" in r.stdout
