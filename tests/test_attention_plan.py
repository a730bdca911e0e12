"""The launch plan of the interleaved attention kernels, replayed on the CPU by tests/plan/driver.cpp from the header that the
kernels use."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_worker_of_a_segment_has_a_part_of_it(tmp_path):
    exe = os.path.join(str(tmp_path), "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", os.path.join(ROOT, "tests", "plan", "driver.cpp"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_09731_amd", "csrc"),
                    "-I", os.path.join(ROCM, "include"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "plan driver ok" in r.stdout, r.stdout + r.stderr
