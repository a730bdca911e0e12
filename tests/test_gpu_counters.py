"""Arrival counters of the attention call that are not zero (as calls of one context that overlap, which its contract excludes,
can leave them) spoil no call beyond the next: each call clears those of the one after it."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2604_09731_amd import binding as B
from tests.test_gpu_tiled_attention import Inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SOURCE = """
#include "common.h"
extern "C" int32_t* counters_of(smart_ctx* c, size_t* n, size_t* plan) {
  *n = c->counters;
  *plan = c->plan_bytes;
  return c->arrive;
}
"""


@pytest.mark.gpu
@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_counters_that_are_not_zero_are_cleared(tmp_path):
    import torch
    (tmp_path / "c.cpp").write_text(SOURCE)
    so = str(tmp_path / "c.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", str(tmp_path / "c.cpp"), "-o", so, "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_09731_amd", "csrc"), "-I",
                    os.path.join(ROCM, "include")], check=True, capture_output=True, text=True)
    counters_of = ctypes.CDLL(so).counters_of
    counters_of.restype = ctypes.c_void_p
    counters_of.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t), ctypes.POINTER(ctypes.c_size_t)]
    lib = B.SmartTree(0)
    # every class, segments of two and more pieces
    # (two calls of one shape in turn: parts that the other left would not be right)
    calls = [Inputs([4, 20, 128, 4, 20, 128], [3000, 2500, 2000, 100, 700, 1500], 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED,
                    seed=seed) for seed in (1, 2)]
    lib.set_option(B.SMART_OPT_TVA_WORKERS, 40)      # (the finishing form: few workgroups for these segments)
    want = [x.run(lib) for x in calls]
    n, plan = ctypes.c_size_t(), ctypes.c_size_t()
    at = counters_of(lib._ctx, ctypes.byref(n), ctypes.byref(plan))
    assert at and n.value >= 6 * 2 * 8
    sets = 3
    ones = torch.ones(sets * n.value, dtype=torch.int32).pin_memory()
    for value in (1, 2, -1):
        ones.fill_(value)
        assert B._lib().tree_upload(lib._ctx, B._stream_ptr(), ones.data_ptr(), at, ones.numel()) == 0
        torch.cuda.synchronize()
        calls[0].run(lib)
        for i in (1, 0, 1, 0, 1):
            assert all(torch.equal(got, ref) for got, ref in zip(calls[i].run(lib), want[i]))
