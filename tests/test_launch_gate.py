"""The admission of kernels whose blocks wait for one another, on host threads."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grids_in_flight_fit_the_device_together(tmp_path):
    exe = str(tmp_path / "launch_gate_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_1311_2719_amd", "csrc"),
                           os.path.join(ROOT, "tests", "launch_gate_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
