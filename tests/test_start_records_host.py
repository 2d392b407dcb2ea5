"""Start records against the items and the block table, for random batches (a C++ program linked with the plan builder alone)."""
import os
import subprocess

from paper_2605_06914_amd.build import CSRC, ROOT


def test_start_records(tmp_path):
    exe = tmp_path / "starts"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(exe),
                    os.path.join(ROOT, "tests", "sanitize", "starts.cpp"), os.path.join(CSRC, "taper_plan.cpp")], check=True, timeout=300)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
