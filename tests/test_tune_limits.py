"""The autotuner's workgroups per CU belong to the plan it chose, not to the
one it timed last (tests/tune_limits.cpp, host code of the library only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2207_06649_amd")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the HIP headers")
def test_blocks_per_cu_of_the_chosen_plan(tmp_path):
    if not os.path.exists(os.path.join(PKG, "libpmbs.so")):
        from paper_2207_06649_amd import build
        build.build()
    exe = str(tmp_path / "limits")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(PKG, "csrc"), "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "tune_limits.cpp"),
                    os.path.join(PKG, "libpmbs.so"), "-Wl,-rpath," + PKG, "-L/opt/rocm/lib",
                    "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
