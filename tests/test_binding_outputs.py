"""The int32 outputs of a binding call are rows of one allocation: each is contiguous and begins where a tensor of its own
would (a multiple of 512 bytes), whatever the lengths."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B


@pytest.mark.parametrize("n", [0, 1, 127, 128, 129, 1000])
@pytest.mark.parametrize("rows", [2, 5])
def test_rows_begin_at_whole_rows(n, rows):
    r = B._i32_rows(rows, n, "cpu")
    assert len(r) == rows
    for i, x in enumerate(r):
        assert x.shape == (n,) and x.is_contiguous()
        assert n == 0 or x.data_ptr() - r[0].data_ptr() == i * ((4 * n + 511) // 512) * 512


@pytest.mark.gpu
@pytest.mark.parametrize("batch,nodes", [(1, 1), (3, 7), (2, 64), (130, 3)])
def test_outputs_of_the_calls_are_aligned(batch, nodes):
    import torch
    lib = B.SmartTree(0)
    N = batch * nodes
    cu = np.arange(batch + 1, dtype=np.int32) * nodes
    parent = np.tile(np.arange(-1, nodes - 1, dtype=np.int32), batch)
    pin = lambda a: torch.from_numpy(a).pin_memory()
    lens = torch.full((batch,), 5, dtype=torch.int32, device="cuda")
    packed = lib.tree_upload_pack(pin(cu), pin(parent), pin(parent), lens)
    d_cu, d_parent, d_token = packed[:3]
    outs = list(packed) + list(lib.tree_pack(d_cu, d_parent, lens))
    length, path, bonus = lib.tree_accept(d_cu, d_parent, d_token, d_token, 4)
    k = torch.randn(N, 2, 64, device="cuda")
    table = torch.arange(batch * 2, dtype=torch.int32, device="cuda").view(batch, 2)
    kc = torch.zeros(batch * 2, 2, 16 * 64, device="cuda")
    outs += [length, path, bonus]
    outs += list(lib.tree_commit(d_cu, length, path, k, k, kc, kc.clone(), table, lens, B.SMART_KV_INTERLEAVED, 16,
                                 batch * 2, kc.stride(0), kc.stride(1)))
    state = B.DeviceLayerState(batch, max(2, nodes), "cuda:0")
    lib.select_begin(state, torch.zeros(batch, dtype=torch.int32, device="cuda"),
                     torch.ones(max(2, nodes) + 2, dtype=torch.float64, device="cuda"))
    for cap in (None, batch * max(2, nodes) + 1, batch * max(2, nodes) + 127):
        compact = lib.tree_compact_pack(state, lens, cap)
        outs += list(compact)
        assert compact[6].shape == (cap if cap else batch * max(2, nodes), 2) and compact[0].shape == (batch + 1,)
        assert compact[7].shape == (batch,) and all(x.shape == compact[1].shape for x in compact[2:6])
    torch.cuda.synchronize()
    for x in outs:
        assert x.data_ptr() % 512 == 0 and x.is_contiguous()
