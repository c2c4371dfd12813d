"""libqs's host code without a device: a native program that defines the HIP
entry points itself loads the built library and drives its C ABI (one process
per case)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_26423_amd")

CASES = ["switched_stream", "same_stream", "no_memory", "many_shots", "many_bins", "deep_batch", "every_plan"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    if not os.path.exists(os.path.join(PKG, "libqs.so")):
        from paper_2604_26423_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("native") / "host_runtime")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "native", "host_runtime.cpp"), "-o", exe, "-L" + PKG, "-l:libqs.so",
                    "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined"], check=True, capture_output=True, text=True)
    return exe


@pytest.mark.parametrize("case", CASES)
def test_host_runtime(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == f"ok {case}\n", r.stdout + r.stderr
