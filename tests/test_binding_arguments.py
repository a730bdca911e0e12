"""Integer arguments of the binding's native calls: what is no integer is refused, as ctypes refuses it, and nothing is called."""
import ctypes
import importlib.machinery
import importlib.util
import os
import shutil

import numpy as np
import pytest
import torch

from paper_2604_09731_amd import binding as B

I32 = torch.zeros(4, dtype=torch.int32)
I64 = torch.zeros(4, dtype=torch.int64)
X = torch.zeros(4, 2, 64)
PATH = torch.zeros(3, 5, dtype=torch.int32)
# name: its arguments (batch of 3, 4 nodes), the positions of those that are integers
CALLS = {
    "rope": ([0, I32, X, X, 1e4, None, 0], [0]),
    "cache_write": ([0, X, X, I64, X, X, 1, 16, 1, 1024, 512, 0, False, None, None], [0, 6, 7, 8, 9, 10, 11]),
    "attention": ([0, X, X, X, X, X, I32.view(2, 2), I32, I32, I64, 0.1, 1, 16, None, None, False, 0, None, None, False, None],
                  [0, 11, 12, 16]),
    "accept": ([0, I32, I32, I32, I32, 4], [0, 5]),
    "sample": ([0, I32, I32, I32, torch.zeros(4, 9), 4, 1, 2], [0, 5]),
    "commit": ([0, I32, I32, PATH, X, X, X, X, I32.view(2, 2), I32, 1, 16, 1, 1024, 512, 0, None, None],
               [0, 10, 11, 12, 13, 14, 15]),
}


@pytest.fixture()
def native(tmp_path):
    """A copy of the module with state of its own, whose entry points count how often they are called."""
    path = shutil.copy(os.path.join(os.path.dirname(B.__file__), "_marshal.so"), tmp_path / "_marshal.so")
    loader = importlib.machinery.ExtensionFileLoader("_marshal", str(path))
    module = importlib.util.module_from_spec(importlib.util.spec_from_loader("_marshal", loader))
    called = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int32)(lambda: called.append(1) or 0)
    address = ctypes.cast(entry, ctypes.c_void_p).value
    module.setup((address,) * len(B._NATIVE_ENTRIES), None, lambda: 0, lambda device: 0)
    return module, called, entry


@pytest.mark.parametrize("name", sorted(CALLS))
def test_integer_arguments(name, native):
    module, called, entry = native          # (entry: kept alive)
    args, integers = CALLS[name]
    call = getattr(module, name)
    call(*args)
    assert len(called) == 1
    for i in integers:
        for wrong in (1.0, 2.5, "1", None):
            with pytest.raises(TypeError):
                call(*args[:i], wrong, *args[i + 1:])
        assert len(called) == 1
        call(*args[:i], np.int64(args[i]), *args[i + 1:])
        assert called.pop() and len(called) == 1
