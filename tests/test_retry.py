"""Host-only check (no GPU) of the buffers of a second attempt whose candidates
overflowed in the first, and of what the next call starts with."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1311_5334_amd", "csrc")


def test_members_of_a_second_attempt(tmp_path):
    exe = str(tmp_path / "retry_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-I" + CSRC,
                           os.path.join(HERE, "native", "retry_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "retry ok" in r.stdout
