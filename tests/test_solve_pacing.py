"""How far ahead of the device a solve queues: the rule alone, and a host that is held up now and
then, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pacing_rule(tmp_path):
    exe = tmp_path / "pace_test"
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                           os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2003_09956_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "pace_test.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all pacing checks passed" in r.stdout, r.stderr
