"""A step whose merges are a launch of their own enqueues two launches that share partial rows: nobody else's launches on the same rows
may come between them, whether another thread calls on the same context and stream or replays a graph.  The host code against a stand-in
for the HIP runtime, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_06914_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")


def test_the_two_launches_of_a_call_stay_together(tmp_path):
    exe = tmp_path / "launch_pairs"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           "-I", SAN, "-I", "/opt/rocm/include", "-o", str(exe), os.path.join(SAN, "launch_pairs.cpp"),
                           os.path.join(SAN, "hip_host.cpp"), os.path.join(CSRC, "taper_api.cpp"), os.path.join(CSRC, "taper_plan.cpp"),
                           os.path.join(CSRC, "taper_admission.cpp"), "-lpthread"])
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok"), run.stdout + run.stderr
