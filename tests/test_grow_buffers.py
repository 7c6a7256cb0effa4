"""Device buffers that grow: after a refused allocation there is neither buffer nor capacity (a call
that needs less than was held before would otherwise go on with a null pointer on the device)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_09956_amd", "csrc")


def test_refused_growth_keeps_no_capacity(tmp_path):
    exe = tmp_path / "grow_test"
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC,
                           os.path.join(ROOT, "tests", "native", "grow_test.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all buffer checks passed" in r.stdout, r.stderr


def test_kept_buffers_grow_nowhere_else():
    """A capacity is only ever set where the buffer is: no allocation into a kept buffer that leaves
    the capacity of the one before it."""
    for name in ("host.hip", "batch.hip"):
        src = open(os.path.join(CSRC, name)).read()
        for buf in ("part", "pdot", "stage", "cert_list"):
            assert not re.search(r"hipMalloc\(&c->%s\b" % buf, src), (name, buf)
