"""Host-only check (no GPU) of the rule that chooses binned cells or line grids
for a call: the faster of the two where both were timed."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1311_5334_amd", "csrc")


def test_cells_or_line_grids(tmp_path):
    exe = str(tmp_path / "few_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", "/opt/rocm/include", "-I" + CSRC,
                           "-I" + os.path.join(ROOT, "include"),
                           os.path.join(HERE, "native", "few_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "few ok" in r.stdout
