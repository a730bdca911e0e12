"""The tiled path's finishing kernel around its limits of one, 128 and 640 groups of eight rows (seven, one or no
wavefronts of a workgroup go through the partials beside the one for the tree part), with one to many partials a row, against
the general kernel; tolerances as in test_gpu_tiled_attention."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B
from tests.test_gpu_tiled_attention import Inputs, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("nodes,workers", [(1, 0), (127, 0), (128, 5), (129, 0), (639, 7), (640, 0), (641, 0), (1025, 0)])
def test_rows_around_the_limits(dtype, D, nodes, workers):
    """Eight query heads: a group of eight rows per node.  A wide table: the split form, however short the prefixes."""
    import torch
    lib = B.SmartTree(0)
    sizes = [1] if nodes == 1 else [nodes % 100] + [100] * (nodes // 100)
    lens = np.random.default_rng(nodes).integers(0, 1500 if nodes < 200 else 200, len(sizes))
    lens[-1] = 1400
    x = Inputs(sizes, lens, 8, 2, D, 16, dtype, B.SMART_KV_PLAIN, seed=nodes, spare_columns=600)
    ref = x.run(lib, general=True)
    lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
    status = torch.full((len(sizes),), -3, dtype=torch.int32, device="cuda")
    got = x.run(lib, status=status)
    assert_close(got, ref)
    assert not status.any()
    again = x.run(lib)
    assert all(torch.equal(p, q) for p, q in zip(got, again))


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 128)])
@pytest.mark.parametrize("workers", [0, 2, 17, 64, 150])
def test_shares_that_begin_behind_a_segments_steps(dtype, D, workers):
    """Segments of no, one and a few steps of one, two and four row tiles, and of two row groups: with enough segments each
    counts more than its steps, and a share may begin where only that is left."""
    import torch
    lib = B.SmartTree(0)
    g = np.random.default_rng(workers)
    sizes = g.choice([1, 8, 9, 17, 33, 60], 40)
    lens = g.choice([0, 1, 64, 65, 128, 129, 300, 700], 40)
    x = Inputs(sizes, lens, 8, 2, D, 16, dtype, B.SMART_KV_PLAIN, seed=workers, spare_columns=600)
    ref = x.run(lib, general=True)
    lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
    got = x.run(lib)
    assert_close(got, ref)
    again = x.run(lib)
    assert all(torch.equal(p, q) for p, q in zip(got, again))
