"""Host-only check (no GPU) of how the counting kernel's items are dealt to its
workgroups: every item to one of them, whatever the sizes. (Two workgroups that
list the same candidate write the same member list at once.)"""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1311_5334_amd", "csrc")


def test_every_item_has_one_taker(tmp_path):
    exe = str(tmp_path / "deal_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", "/opt/rocm/include", "-I" + CSRC,
                           os.path.join(HERE, "native", "deal_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "deal ok" in r.stdout
