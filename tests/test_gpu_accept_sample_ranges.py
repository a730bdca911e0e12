"""tree_accept_sample where the kernels change shape: vocabularies on both sides of 512 tokens per range (8 or 32 tokens
per lane in the bonus search, several pieces), batches on both sides of 128 rows (one or four ranges per wavefront), trees
with more nodes than are fetched ahead; bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import accept_sample as A
from paper_2604_09731_amd import binding as B
from tests.test_gpu_accept_sample import _case, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,sizes", [(32768, [5, 1]), (32769, [9, 8]), (131076, [4, 2]), (263, [7, 9, 64, 40, 7]),
                                     (264, [8, 9, 64, 40, 8]), (513, [128, 1])])
@pytest.mark.parametrize("pad", [0, 1])
def test_ranges_and_rows(V, sizes, pad):
    import torch
    lib = B.SmartTree(0)
    cu, parent, token, prob = _case(V + pad, sizes, V)
    prob[0, :3] = (0.0, -1.0, np.nan)                     # weights of zero
    prob[-1, -1] = 1.5                                    # counts as 1
    wide = torch.full((prob.shape[0], V + pad), 7.0, dtype=torch.float32, device="cuda")
    wide[:, :V] = _dev(prob)
    for seed, step in ((3, 1), (5, 2 ** 35), (2 ** 60, 9)):
        got = lib.tree_accept_sample(_dev(cu), _dev(parent), _dev(token), wide[:, :V], 8, seed, step)
        torch.cuda.synchronize()
        assert tuple(x.cpu().numpy().tolist() for x in got) == tuple(A.accept_sample(cu, parent, token, prob, seed, step, 8))
