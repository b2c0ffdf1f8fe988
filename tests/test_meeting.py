"""The words through which the workgroups of a launch meet (csrc/meeting.h), compiled for the host: threads in their place, waits of a few polls."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workgroups_that_give_up_take_all_along(tmp_path):
    exe = str(tmp_path / "meeting_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(ROOT, "paper_2301_07482_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "meeting_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, "3000"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
