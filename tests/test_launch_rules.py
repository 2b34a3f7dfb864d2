"""CPU test of the rules that choose and size launches (internal.h): compiled for the host and checked over
small and large operands, among them ones larger than any device memory."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_launch_rules(tmp_path):
    exe = str(tmp_path / "rules")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
           f"-I{os.path.join(ROOT, 'paper_1507_08101_amd', 'csrc')}",
           os.path.join(ROOT, "tests", "sanitize", "launch_rules_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "launch rules ok" in r.stdout, r.stderr[-3000:]
