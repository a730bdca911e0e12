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


SETS = 3
needs_compiler = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def counters_of(tmp_path_factory):
    """(context) -> address of its counters, of one set."""
    where = tmp_path_factory.mktemp("counters")
    (where / "c.cpp").write_text(SOURCE)
    so = str(where / "c.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", str(where / "c.cpp"), "-o", so, "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_09731_amd", "csrc"), "-I",
                    os.path.join(ROCM, "include")], check=True, capture_output=True, text=True)
    entry = ctypes.CDLL(so).counters_of
    entry.restype = ctypes.c_void_p
    entry.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t), ctypes.POINTER(ctypes.c_size_t)]

    def of(lib):
        n, plan = ctypes.c_size_t(), ctypes.c_size_t()
        return entry(lib._ctx, ctypes.byref(n), ctypes.byref(plan)), n.value
    return of


def fill(lib, at, n, value):
    import torch
    values = torch.full((n,), value, dtype=torch.int32).pin_memory()
    assert B._lib().tree_upload(lib._ctx, B._stream_ptr(), values.data_ptr(), at, n) == 0
    torch.cuda.synchronize()


@needs_compiler
@pytest.mark.gpu
def test_counters_that_are_not_zero_are_cleared(counters_of):
    import torch
    lib = B.SmartTree(0)
    # every class, segments of two and more pieces
    # (two calls of one shape in turn: parts that the other left would not be right)
    calls = [Inputs([4, 20, 128, 4, 20, 128], [3000, 2500, 2000, 100, 700, 1500], 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED,
                    seed=seed) for seed in (1, 2)]
    lib.set_option(B.SMART_OPT_TVA_WORKERS, 40)      # (the finishing form: few workgroups for these segments)
    want = [x.run(lib) for x in calls]
    at, n = counters_of(lib)
    assert at and n >= 6 * 2 * 8
    for value in (1, 2, -1):
        fill(lib, at, SETS * n, value)
        calls[0].run(lib)
        for i in (1, 0, 1, 0, 1):
            assert all(torch.equal(got, ref) for got, ref in zip(calls[i].run(lib), want[i]))


@needs_compiler
@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True])
def test_a_call_of_few_workers_clears_the_whole_set(fp8, counters_of):
    """The workgroups of a small call that have no share of its work clear theirs of the counters all the same."""
    import torch
    lib = B.SmartTree(0)
    few = Inputs([3], [40], 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=1)
    many = Inputs([4, 20, 40, 12] * 10, [3000, 2500, 2000, 1500] * 10, 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=2)
    want = many.run(lib)
    at, n = counters_of(lib)
    assert at and n >= 40 * 2 * 8
    for value in (1, 2, -1):
        fill(lib, at, SETS * n, value)
        few.run(lib)
        assert all(torch.equal(got, ref) for got, ref in zip(many.run(lib), want))
