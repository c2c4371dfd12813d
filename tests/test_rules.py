"""Rules by which the library picks a way of computing, checked on the host over
their whole range (tests/native/rules.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules(tmp_path):
    exe = str(tmp_path / "rules")
    b = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "paper_2604_26423_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "rules.cpp"), "-o", exe], capture_output=True, text=True)
    if b.returncode != 0 and "hip_runtime.h" in b.stderr:
        pytest.skip("HIP headers not usable by the host compiler here")
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
