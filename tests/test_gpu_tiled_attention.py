"""The tiled matrix-core attention path (every type, layout, head dim and block size besides bf16 / interleaved /
128 / 16) against the general kernel, which walks the keys of one row at a time in fp32, over the forms both accept,
with prefixes of up to 700 keys; and against the oracle in 64 bits with prefixes of up to 2500.

Tolerances.  fp32: both sides sum the same products in binary32 in different orders; a dot product of D <= 128
terms and a weighted sum of the keys move by a few 1e-7 of the output's scale, the repository's 1e-5 bounds
them.  bf16: both sides hold scores, probabilities and sums in binary32 (the tiled path splits a probability into three
bf16 values, exactly), so the outputs differ where a binary32 difference of that size crosses a rounding boundary:
one bf16 unit, 2^-7 of the element at most.  lse: fp32 on both sides, |lse| < 16."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B
from paper_2604_09731_amd import workloads as W

pytestmark = pytest.mark.gpu

ROW_SIZES = [1, 31, 32, 33, 64, 65, 127, 128]        # nodes; at G = 1 rows: edges of the 32-row tiles and 128-row groups


@pytest.fixture(scope="module")
def lib():
    return B.SmartTree(0)


class Inputs:
    def __init__(self, sizes, lens, Hq, Hkv, D, bs, dtype, layout, fp8=False, pad=0, seed=3, spare_columns=1):
        import torch
        g = np.random.default_rng(seed)
        t = lambda a, dt=None: torch.from_numpy(np.ascontiguousarray(a, dt)).cuda()
        self.layout, self.bs, self.D = layout, bs, D
        sizes, lens = np.asarray(sizes), np.asarray(lens)
        self.cu_host = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        N = int(self.cu_host[-1])
        self.parent = t(np.concatenate([W.random_tree(int(n), g) for n in sizes]), np.int32)
        self.cu, self.len = t(self.cu_host), t(lens, np.int32)
        blocks = (lens + bs - 1) // bs
        nb = int(blocks.sum()) + 2
        perm = g.permutation(nb)
        table = np.full((len(sizes), max(1, int(blocks.max())) + spare_columns), -1, np.int32)
        at = 0
        for b, m in enumerate(blocks):
            table[b, :m] = perm[at:at + m]
            at += int(m)
        self.table = t(table)
        tdt = torch.float32 if dtype == "f32" else torch.bfloat16
        rnd = lambda *s: t(g.standard_normal(s, dtype=np.float32)).to(tdt)
        self.q, self.k_tree, self.v_tree = rnd(N, Hq, D), rnd(N, Hkv, D), rnd(N, Hkv, D)
        self.kw = dict(k_scale=0.05, v_scale=0.25) if fp8 else {}
        owned = np.zeros((nb, bs), bool)
        for b, m in enumerate(lens):
            for i in range(int(m)):
                owned[table[b, i // bs], i % bs] = True
        caches = []
        for _ in range(2):
            x = g.standard_normal((nb, Hkv, bs, D), dtype=np.float32) * (20 if fp8 else 1)
            x[~owned[:, None, :].repeat(Hkv, 1)] = np.nan                      # nothing may read an unowned slot
            x = t(x)
            x = x.clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else x.to(tdt)
            caches.append(x)
        k, v = caches
        self.plain = [c.view(torch.float8_e4m3fn).float() * self.kw[s] if fp8 else c.float()
                      for c, s in zip(caches, ("k_scale", "v_scale"))]             # [block, kv head, slot, head dim]
        if layout == B.SMART_KV_INTERLEAVED:
            k = k.reshape(nb, Hkv, bs, D // 8, 8).permute(0, 1, 3, 2, 4).reshape(nb, Hkv, 1, bs * D)
            v = v.reshape(nb, Hkv, bs // 8, 8, D).permute(0, 1, 2, 4, 3).reshape(nb, Hkv, 1, bs * D)
        # pad: rows, pages and blocks further apart than they are long
        def spread(c):
            big = torch.zeros((c.shape[0], c.shape[1] + (1 if pad else 0), c.shape[2], c.shape[3] + pad), dtype=c.dtype, device="cuda")
            view = big[:, :c.shape[1], :, :c.shape[3]]
            view.copy_(c)
            return view
        self.k, self.v = spread(k), spread(v)

    def run(self, lib, general=False, static=False, cu=None, table=None, status=None, out=None):
        import torch
        _, _, _, mask, _ = lib.tree_pack(self.cu, self.parent, self.len)
        lib.set_option(B.SMART_OPT_TVA_FORCE_GENERAL, int(general))
        try:
            r = lib.tree_verify_attention(self.q, self.k_tree, self.v_tree, self.k, self.v,
                                          self.table if table is None else table, self.len, self.cu if cu is None else cu,
                                          mask, 1.0 / np.sqrt(self.D), self.layout, block_size=self.bs, want_lse=True,
                                          static=static, status=status, out=out, **self.kw)
        finally:
            lib.set_option(B.SMART_OPT_TVA_FORCE_GENERAL, 0)
        torch.cuda.synchronize()
        return r


def assert_close(got, ref):
    import torch
    for x, y in zip(got, ref):
        x, y = x.double(), y.double()
        assert torch.equal(torch.isinf(x), torch.isinf(y))
        assert not torch.isnan(x).any()
        fin = torch.isfinite(y)
        if not fin.any():
            continue
        tol = 1e-5 * max(1.0, float(y[fin].abs().max()))
        if got[0].dtype == torch.bfloat16 and x.ndim == 3:
            assert bool(((x - y).abs() <= tol + 2.0 ** -7 * y.abs()).all())
        else:
            assert float((x - y)[fin].abs().max()) <= tol


FORMS = [(dt, fp8, lay, D) for dt in ("f32", "bf16") for fp8 in (False, True)
         for lay in (B.SMART_KV_PLAIN, B.SMART_KV_INTERLEAVED) for D in (64, 128)]


@pytest.mark.parametrize("dtype,fp8,layout,D", FORMS)
def test_every_form_equals_the_general_kernel(lib, dtype, fp8, layout, D):
    """Tile, step and row-group edges: lengths around 16, 32, 64, 128 keys, tree sizes around 32 and 128 rows, block
    sizes that do and do not divide a tile; the split and the workspace-free form."""
    lens = [0, 1, 15, 17, 64, 65, 127, 300]
    for bs, Hq, Hkv, pad in ((8, 3, 3, 0), (24, 8, 2, 8), (64, 7, 1, 16)):
        x = Inputs(ROW_SIZES, lens, Hq, Hkv, D, bs, dtype, layout, fp8, pad=pad if layout == B.SMART_KV_PLAIN else 0)
        ref = x.run(lib, general=True)
        assert_close(x.run(lib), ref)
        assert_close(x.run(lib, static=True), ref)


@pytest.mark.parametrize("batch", [1, 64, 65, 130, 512, 513, 1100])
@pytest.mark.parametrize("workers", [0, 1, 3])
def test_batches_and_shares(lib, batch, workers):
    """Batches around the 64 sequences one scan holds and the 512 that every wavefront scans for itself, empty trees and
    prefixes among them; shares of one worker that run over many segments; the workspace-free form."""
    g = np.random.default_rng(batch)
    sizes, lens = g.integers(0, 9, batch), g.integers(0, 260, batch)
    sizes[0] = 5
    x = Inputs(sizes, lens, 8, 2, 64, 16, "f32", B.SMART_KV_PLAIN)
    lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
    try:
        ref = x.run(lib, general=True)
        assert_close(x.run(lib), ref)
        assert_close(x.run(lib, static=True), ref)
    finally:
        lib.set_option(B.SMART_OPT_TVA_WORKERS, 0)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("batch", [3, 600])
def test_rows_nobody_owns_around_the_trees(lib, static, batch):
    """Rows before the first and behind the last range, of a range longer than a tree, of one that leaves the arrays."""
    import torch
    x = Inputs([2] * (batch - 2) + [100, 52], [17, 0, 70] * (batch // 3), 8, 2, 64, 16, "f32", B.SMART_KV_PLAIN)
    N = int(x.cu_host[-1])
    inside, shifted, beyond, longer = (x.cu_host.copy() for _ in range(4))
    inside[0], inside[-2:] = 1, [N - 60, N - 9]
    shifted[:2] = -1, 1
    beyond[-1] = N + 1
    longer[-2] = N - 2                          # 150 nodes: 128 of them are served
    for cu in (x.cu_host, inside, shifted, beyond, longer):
        cu = torch.tensor(cu, dtype=torch.int32, device="cuda")
        ref = x.run(lib, general=True, cu=cu, out=torch.full_like(x.q, 7.0))
        assert_close(x.run(lib, cu=cu, static=static, out=torch.full_like(x.q, 7.0)), ref)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_what_the_general_kernel_does_with_odd_inputs(lib, static, dtype):
    import torch
    x = Inputs([5, 20, 70, 3, 9], [100, 333, 64, 0, 50], 8, 2, 128, 16, dtype, B.SMART_KV_PLAIN)
    # rows past the trees (total_nodes as a capacity) and ranges that leave the arrays: zero, lse -inf
    N = int(x.cu_host[-1])
    for bad in (x.cu_host - [0, 0, 0, 0, 0, 9], [0, 5, 25, 95, 98, N + 4], [-1, 5, 25, 95, 98, N], [N + 1] * 6):
        cu = torch.tensor(np.asarray(bad), dtype=torch.int32, device="cuda")
        ref = x.run(lib, general=True, cu=cu, out=torch.full_like(x.q, 7.0))
        assert_close(x.run(lib, cu=cu, static=static, out=torch.full_like(x.q, 7.0)), ref)
    # block-table entries outside the cache: read as the nearest block, reported
    table = x.table.clone()
    table[1, 3], table[2, 3], table[0, 7] = -5, 10 ** 6, 10 ** 6
    table[x.table < 0] = -9
    status = [torch.full((5,), 77, dtype=torch.int32, device="cuda") for _ in range(2)]
    x.k.nan_to_num_(0.0)
    x.v.nan_to_num_(0.0)
    ref = x.run(lib, general=True, table=table, status=status[0])
    assert_close(x.run(lib, table=table, status=status[1], static=static), ref)
    assert status[0].tolist() == status[1].tolist() == [0, 1, 1, 0, 0]
    # what one node holds reaches only the nodes below it; infinite scores
    x = Inputs([40], [90], 8, 2, 128, 16, dtype, B.SMART_KV_PLAIN)
    x.v_tree[39] = float("nan")
    x.k_tree[38] = float("inf")
    x.q[37, 0] = float("-inf")
    x.k[int(x.table[0, 2]), 1, 3] = float("inf")
    got, ref = x.run(lib, static=static), x.run(lib, general=True)
    for a, b in zip(got, ref):
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        both = torch.isfinite(a) & torch.isfinite(b)
        assert torch.equal(torch.isfinite(a), torch.isfinite(b)) and both.any()


def test_unaligned_rows_run_the_general_kernel(lib):
    """Strides that put rows off the 16-byte chunks the tiled path loads: the same call, the general kernel's bits."""
    import torch
    x = Inputs([9, 30], [100, 77], 8, 2, 64, 16, "bf16", B.SMART_KV_PLAIN, pad=2)
    a, b = x.run(lib), x.run(lib, general=True)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_a_captured_call_holds_no_workspace(lib):
    """A graph of the call stays right after a larger call has replaced the context's workspace."""
    import torch
    own = B.SmartTree(0)
    x = Inputs([9, 30, 4], [400, 77, 129], 8, 2, 64, 16, "f32", B.SMART_KV_PLAIN)
    _, _, _, mask, _ = own.tree_pack(x.cu, x.parent, x.len)
    out = torch.empty_like(x.q)
    call = lambda: own.tree_verify_attention(x.q, x.k_tree, x.v_tree, x.k, x.v, x.table, x.len, x.cu, mask, 0.125, x.layout,
                                             block_size=16, out=out)
    call()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    big = Inputs([100] * 70, [40] * 70, 8, 2, 128, 16, "bf16", B.SMART_KV_PLAIN)
    ref = x.run(own, general=True)[0]
    for _ in range(3):
        big.run(own)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert_close((out,), (ref,))


def test_a_graph_of_the_interleaved_kernel_keeps_its_workspace(lib):
    """Eager calls of this path grow a buffer of their own: a captured call of the interleaved bf16 kernel, which holds the
    context's workspace, replays to the same bits between them.  One of them grows while the capture is under way."""
    import torch
    own = B.SmartTree(0)
    x = Inputs([9, 30, 4], [400, 77, 129], 8, 2, 128, 16, "bf16", B.SMART_KV_INTERLEAVED)
    big = [Inputs([100] * n, [600] * n, 8, 2, 128, 16, "bf16", B.SMART_KV_PLAIN) for n in (3, 20, 70)]
    refs = [b.run(lib, general=True) for b in big]
    _, _, _, mask, _ = own.tree_pack(x.cu, x.parent, x.len)
    big_mask = own.tree_pack(big[0].cu, big[0].parent, big[0].len)[3]
    out, big_out = torch.empty_like(x.q), torch.empty_like(big[0].q)
    def call(i, m, o):
        own.tree_verify_attention(i.q, i.k_tree, i.v_tree, i.k, i.v, i.table, i.len, i.cu, m, 1 / np.sqrt(128), i.layout,
                                  block_size=16, out=o)
    call(x, mask, out)
    torch.cuda.synchronize()
    ref = out.clone()
    other = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, mask, out)
        with torch.cuda.stream(other):
            call(big[0], big_mask, big_out)
    torch.cuda.synchronize()
    assert_close((big_out,), (refs[0][0],))
    for b, r in zip(big, refs):
        assert_close(b.run(own), r)
        junk = torch.full((1 << 24,), float("nan"), device="cuda")      # what a freed workspace would be handed out as
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        del junk


@pytest.mark.parametrize("dtype,longest,rows", [("bf16", 512, 64), ("bf16", 128, 384), ("f32", 64, 384)])
def test_around_the_one_launch_rule(lib, dtype, longest, rows):
    """Small trees on tables that hold at most, and just more than, what one workgroup per segment takes; a mean of as many
    rows as the rule takes and one above it."""
    n = rows // 4
    for sizes in ([n, n], [n, n + 1], [1, 2 * n - 1 if n < 64 else 128]):
        for extra in (0, 1):
            x = Inputs(sizes, [longest, 5], 8, 2, 64, 16, dtype, B.SMART_KV_PLAIN, spare_columns=extra)
            assert_close(x.run(lib), x.run(lib, general=True))


def _value_column(x, b, token, g, d):
    """The view of one cached value (whatever the layout): x.v[page, g, ...] of sequence b's token, head dim d."""
    page, slot = int(x.table[b, token // x.bs]), token % x.bs
    if x.layout == B.SMART_KV_PLAIN:
        return x.v[page, g, slot, d:d + 1]
    at = ((slot // 8) * x.D + d) * 8 + slot % 8
    return x.v[page, g, 0, at:at + 1]


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("layout", [B.SMART_KV_PLAIN, B.SMART_KV_INTERLEAVED])
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64)])
def test_infinite_cached_values(lib, static, layout, dtype, D):
    """p times an infinite value is that infinity for every p > 0; opposite infinities in one head dim and NaN give NaN.
    In the first, an inner and the last (ragged) step, for one and for several row tiles."""
    import torch
    inf = float("inf")
    bs = 16 if D == 64 else 8
    x = Inputs([40, 9, 3], [700, 333, 40], 8, 2, D, bs, dtype, layout)
    for b, token, g, d, value in ((0, 3, 0, 5, inf), (0, 300, 1, 6, -inf), (0, 699, 0, 63, inf), (1, 0, 1, 0, -inf),
                                  (1, 332, 0, 33, inf), (1, 10, 0, 17, inf), (1, 200, 0, 17, -inf), (2, 39, 0, 1, -inf),
                                  (2, 7, 1, 40, float("nan")), (2, 8, 1, 41, inf)):
        _value_column(x, b, token, g, d).fill_(value)
    (out, lse), (ref, ref_lse) = x.run(lib, static=static), x.run(lib, general=True)
    assert bool(torch.isposinf(ref).any()) and bool(torch.isneginf(ref).any()) and bool(torch.isnan(ref).any())
    for test in (torch.isposinf, torch.isneginf, torch.isnan):
        assert torch.equal(test(out), test(ref))
    fin = torch.isfinite(ref)
    assert_close((torch.where(fin, out, 0), lse), (torch.where(fin, ref, 0), ref_lse))


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("layout", [B.SMART_KV_PLAIN, B.SMART_KV_INTERLEAVED])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("nodes", [3, 30, 64])
def test_values_near_the_end_of_the_range(lib, static, layout, dtype, nodes):
    """Values of 2^118 whose weighted sum stays below 2^128 as long as no weight exceeds 1, under scores that rise by less
    than the step in which the reference follows the maximum.  (One worker: all steps of a segment in one piece.)"""
    import torch
    x = Inputs([nodes], [512], 2, 1, 64, 16, dtype, layout)
    x.q.fill_(1.0)
    x.k_tree.zero_()
    x.v_tree.fill_(2.0 ** 118)
    x.v.fill_(2.0 ** 118)
    for token in range(512):                     # score 0, then 5 (D k / sqrt(D))
        page, slot = int(x.table[0, token // 16]), token % 16
        k = x.k[page, 0] if layout == B.SMART_KV_PLAIN else x.k[page, 0, 0].view(8, 16, 8).transpose(0, 1)
        k[slot] = 0.0 if token < 128 else 0.625
    lib.set_option(B.SMART_OPT_TVA_WORKERS, 1)
    try:
        got, ref = x.run(lib, static=static), x.run(lib, general=True)
    finally:
        lib.set_option(B.SMART_OPT_TVA_WORKERS, 0)
    assert bool(torch.isfinite(ref[0]).all())
    assert_close(got, ref)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,fp8,layout", [("bf16", False, B.SMART_KV_PLAIN), ("f32", True, B.SMART_KV_INTERLEAVED),
                                              ("f32", False, B.SMART_KV_PLAIN), ("bf16", True, B.SMART_KV_INTERLEAVED)])
def test_offsets_that_are_not_ascending(lib, static, dtype, fp8, layout):
    """Overlapping ranges, more segments than the rows were counted for, descending offsets, batches on both sides of 64:
    every row has the one owner that the general kernel finds, and its value."""
    import torch
    g = np.random.default_rng(4)
    for sizes, lens, offsets in (([5, 20, 70, 3, 9], [100, 333, 64, 0, 50], [0, 25, 5, 95, 98, 107]),
                                 ([2] * 64, list(g.integers(0, 90, 64)), [0, 128] * 32 + [0]),
                                 ([2] * 65, list(g.integers(0, 90, 65)), list(range(130, -1, -2))),
                                 ([2] * 600, list(g.integers(0, 90, 600)), list(range(0, 800, 2)) + list(range(700, 1101, 2))),
                                 ([30, 40], [70, 90], [40, 0, 70]), ([30, 40], [70, 90], [50, -3, 70])):
        x = Inputs(sizes, lens, 8, 2, 64, 8, dtype, layout, fp8)
        cu = torch.tensor(offsets, dtype=torch.int64).to(torch.int32).cuda()
        ref = x.run(lib, general=True, cu=cu, out=torch.full_like(x.q, 7.0))
        assert_close(x.run(lib, cu=cu, static=static, out=torch.full_like(x.q, 7.0)), ref)


@pytest.mark.parametrize("dtype,fp8,layout,D", FORMS)
def test_every_form_equals_the_oracle_on_long_prefixes(lib, oracle_attention, dtype, fp8, layout, D):
    """Many steps per piece and many pieces per segment, in the split and the workspace-free form.  The weighted mean of |V|
    (the oracle's result for |V|) is what rounding errors of scores and sums are relative to: 1e-5 of it; a bf16 output is
    rounded once more, by at most 2^-8 of it (8 significant bits)."""
    import torch
    bs = 8 if layout == B.SMART_KV_INTERLEAVED else (24 if D == 64 else 16)     # (interleaved 128 / 16 is the other path's)
    x = Inputs([9, 40, 3, 64], [2500, 1301, 700, 5], 8, 2, D, bs, dtype, layout, fp8)
    n = lambda t: np.ascontiguousarray(t.float().cpu().numpy())
    def oracle(f):
        k, v = x.plain
        return oracle_attention.tree_attention(n(x.q), n(x.k_tree), f(n(x.v_tree)), n(k), f(n(v)), x.table.cpu().numpy(),
                                               x.len.cpu().numpy(), x.cu_host, x.parent.cpu().numpy(), 1.0 / np.sqrt(D))
    ref, ref_lse = oracle(lambda a: a)
    bound = 1e-5 * oracle(np.abs)[0] + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    for static in (False, True):
        out, lse = x.run(lib, static=static)
        assert (np.abs(out.double().cpu().numpy() - ref) <= bound).all()
        assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 2e-5
