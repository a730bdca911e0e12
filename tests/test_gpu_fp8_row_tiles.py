"""fp8 cache, trees around one and two row tiles of 32 rows per kv head: batches whose mean size and table pick the kernel
that gives both row tiles of a long piece to every wavefront (and those of a short one to a half of the workgroup each),
and batches that run the kernel with halves only; against the general kernel, which holds probabilities in binary32.

Tolerance, element by element.  bf16 has 8 significant bits, so rounding to it moves a number by at most u = 2^-8 of
itself.  The matrix-core path rounds each probability (the row sums are of the unrounded ones), which moves an output by
at most u times the weighted mean of |V| -- the general kernel's result for |V|, itself rounded once -- and both sides
round the output once: u (spread (1 + u) + 2 |ref| (1 + u)).  Binary32 sums and exponentials in another order add a few
1e-6 of the weighted mean (2^-16 covers them)."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B
from tests.test_gpu_tiled_attention import Inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[8, 9, 16, 17], [12, 16, 16, 9], [1, 1, 1, 12], [1, 2, 1, 16, 1, 1]])
@pytest.mark.parametrize("workers", [0, 1, 4, 5])
def test_one_and_two_row_tiles(sizes, workers):
    """G = 4: 32, 33 .. 64 and 65 rows; long shares of one worker (several chunks of 64 tiles per wavefront), pieces around
    the 72 tiles from which on they go as pairs, shares shorter than a wavefront's turn, ragged ends and an empty prefix."""
    import torch
    lib = B.SmartTree(0)
    lens = {1: [20000, 33, 517, 0, 64, 1], 4: [2303, 9001, 2272, 2273, 95, 2400]}.get(workers, [1, 2049, 700, 33, 95, 31])[:len(sizes)]
    x = Inputs(sizes, lens, 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8=True, seed=len(sizes) + workers)
    ref, ref_lse = x.run(lib, general=True)
    v, v_tree = x.v, x.v_tree
    x.v, x.v_tree = v & 0x7F, v_tree.abs()
    spread = x.run(lib, general=True)[0].double()
    x.v, x.v_tree = v, v_tree
    u = 2.0 ** -8
    bound = (u * (1 + u) + 2.0 ** -16) * spread + 2 * u * (1 + u) * ref.double().abs()
    lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
    for static in (False, True):
        out, lse = x.run(lib, static=static)
        assert torch.isfinite(out.float()).all()
        assert bool(((out.double() - ref.double()).abs() <= bound).all())
        assert float((lse - ref_lse).abs().max()) <= 1e-3
        again, again_lse = x.run(lib, static=static)         # states are merged in a fixed order: the same bits every time
        assert torch.equal(again, out) and torch.equal(again_lse, lse)
