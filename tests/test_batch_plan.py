"""How a batch is cut into work items, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan(tmp_path):
    exe = tmp_path / "plan_test"
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-I", os.path.join(ROOT, "paper_2003_09956_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "plan_test.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all plan checks passed" in r.stdout, r.stderr
