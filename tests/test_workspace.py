"""What the library allocates for attention calls, on the CPU: tests/workspace/driver.cpp stands in for the HIP runtime,
counts allocations and launches and lets them fail (no kernel runs)."""
import os
import shutil
import subprocess

import pytest

from paper_2604_09731_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_attention_workspace(tmp_path):
    exe = os.path.join(str(tmp_path), "driver")
    lib = os.path.abspath(B.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unused-result", os.path.join(ROOT, "tests", "workspace", "driver.cpp"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"), lib,
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64", f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "workspace driver ok" in r.stdout, r.stdout + r.stderr
