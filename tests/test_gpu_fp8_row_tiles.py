"""fp8 cache, trees around one and two row tiles of 32 rows per kv head: batches whose mean size picks the kernel that
gives both row tiles to every wavefront, and batches whose mean picks the one that gives one to each half of the
workgroup; against the general kernel, which holds probabilities in binary32.  Tolerance: the matrix-core path rounds a
probability to bf16 (2^-9 of it) and so moves an output by at most 2^-9 of the largest value; both round the output once
more (2^-9 of it): 2e-2 of the output's scale bounds that."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B
from tests.test_gpu_tiled_attention import Inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[8, 9, 16, 17], [12, 16, 16, 9], [1, 1, 1, 12], [1, 2, 1, 16, 1, 1]])
@pytest.mark.parametrize("workers", [0, 1, 5])
def test_one_and_two_row_tiles(sizes, workers):
    """G = 4: 32, 33 .. 64 and 65 rows; long shares of one worker (several chunks of 64 tiles per wavefront), shares
    shorter than a wavefront's turn, ragged ends and an empty prefix."""
    import torch
    lib = B.SmartTree(0)
    lens = ([1, 2049, 700, 33, 95, 31] if workers != 1 else [20000, 33, 517, 0, 64, 1])[:len(sizes)]
    x = Inputs(sizes, lens, 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8=True, seed=len(sizes) + workers)
    ref, ref_lse = x.run(lib, general=True)
    lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
    for static in (False, True):
        out, lse = x.run(lib, static=static)
        assert torch.isfinite(out.float()).all()
        assert float((out.double() - ref.double()).abs().max()) <= 2e-2 * float(ref.double().abs().max())
        assert float((lse - ref_lse).abs().max()) <= 1e-3
