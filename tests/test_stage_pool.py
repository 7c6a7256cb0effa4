"""The server's staging memory: no event is asked or waited for after the stream it was recorded on has
gone (the runtime looks at that stream, and a closed server left an error for the next caller)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_09956_amd", "csrc")


def test_stage_pool(tmp_path):
    exe = tmp_path / "stage_test"
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                           os.path.join(ROOT, "tests", "native", "stage_test.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all staging checks passed" in r.stdout, r.stderr


def test_server_ends_a_stream_in_the_pool_first():
    """Every stream of a request that the server destroys has been ended in the pool before."""
    src = open(os.path.join(CSRC, "server.hip")).read()
    assert len(re.findall(r"hipStreamDestroy\(r\.stream\)", src)) == 1
    assert re.search(r"stages\.end_stream\(r\.stream\);\s*\(void\)hipStreamDestroy\(r\.stream\);", src)
    # the streams of the server's own outlive the pool
    close = src[src.index("void modap_server_destroy("):]
    assert close.index("stages.destroy()") < close.index("hipStreamDestroy(")
