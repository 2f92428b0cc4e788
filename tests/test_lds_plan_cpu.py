"""The LDS layout of an exploration's first levels (host C++, shared with the
library through its header), built with g++ and checked by
tests/lds_plan_check.cpp."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1801_05857_amd", "csrc")


def test_lds_plan(tmp_path):
    exe = tmp_path / "lds_plan_check"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(exe),
                           os.path.join(HERE, "lds_plan_check.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
