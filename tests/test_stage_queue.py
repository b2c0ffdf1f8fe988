"""The queue that hands the stages of transposes to launches (csrc/stage_queue.h), compiled for the host and driven over every order."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_stage_is_handed_out_once_and_the_queue_ends(tmp_path):
    exe = str(tmp_path / "stage_queue_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2301_07482_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "stage_queue_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
