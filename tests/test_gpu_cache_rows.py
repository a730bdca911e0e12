"""kv_cache_write over token runs: prompts that start anywhere in the token list, runs broken by skipped and
out-of-range slots, permuted single tokens, tails shorter than a slot group; every type and layout, byte for byte."""
import numpy as np
import pytest

from oracle import fp8 as F
from oracle import kv_layout as KL
from paper_2604_09731_amd import binding as B
from paper_2604_09731_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _slots(kind, n, bs, nb, rng):
    if kind == "prompts":        # ragged prompts in permuted blocks
        perm, out, at = rng.permutation(nb), [], 0
        while len(out) < n:
            m = int(rng.integers(1, 3 * bs))
            out += [int(perm[(at + i // bs) % nb]) * bs + i % bs for i in range(m)]
            at += (m + bs - 1) // bs
        return np.array(out[:n], np.int64)
    if kind == "offset":         # one run that starts inside a slot group
        return np.arange(3, 3 + n, dtype=np.int64) % (nb * bs)
    if kind == "reversed":
        return np.arange(n, dtype=np.int64)[::-1].copy()
    s = np.arange(n, dtype=np.int64)                       # "holes"
    s[rng.integers(0, n, max(1, n // 9))] = -1
    s[rng.integers(0, n, max(1, n // 20))] = nb * bs + 5
    return s


def _check(dtype, fp8, layout, kind, sizes):
    import torch
    lib = B.SmartTree(0)
    rng = np.random.default_rng(5)
    for n, Hkv, D, bs in sizes:
        nb = 2 * n // bs + 60
        k_src, v_src = (W._normal(1, i, (n, Hkv, D), 1.0, dtype) for i in (1, 2))
        slots = _slots(kind, n, bs, nb, rng)
        keep = {}
        for t, s in enumerate(slots):                       # a slot named twice: no defined winner, so name it once
            if 0 <= s < nb * bs and s in keep:
                slots[t] = -1
            keep[s] = t
        f = lambda x: (W.bf16_bits_to_f32(x) if dtype == "bf16" else x).astype(np.float32)
        val = [F.encode(f(x) / np.float32(sc)) for x, sc in ((k_src, 0.03), (v_src, 0.011))] if fp8 else [k_src, v_src]
        plain = [np.zeros((nb, Hkv, bs, D), v.dtype) for v in val]
        for t, s in enumerate(slots):
            if 0 <= s < nb * bs:
                for p, v in zip(plain, val):
                    p[s // bs, :, s % bs] = v[t]
        tk, tv = H.torch_elems(k_src, dtype, "cuda"), H.torch_elems(v_src, dtype, "cuda")
        cdt = torch.uint8 if fp8 else tk.dtype
        pad = 8 * D                                          # pages and blocks further apart than they are long
        big = [torch.zeros((nb, Hkv + 1, bs * D + pad), dtype=cdt, device="cuda") for _ in range(2)]
        kc, vc = big
        args = (torch.from_numpy(slots).cuda(), kc, vc, layout, bs, nb, kc.stride(0), kc.stride(1))
        if fp8:
            lib.kv_cache_write_fp8(tk, tv, *args, 0.03, 0.011, token_stride=D)
        else:
            lib.kv_cache_write(tk, tv, *args, token_stride=D)
        for c, p, which in zip(big, plain, "kv"):
            got = c.cpu()
            got = (got if fp8 else got.view(torch.int16 if dtype == "bf16" else torch.float32)).numpy().view(p.dtype)
            want = p.reshape(nb, Hkv, bs * D) if layout == B.SMART_KV_PLAIN else KL.interleave_plain_cache(p, which)
            assert np.array_equal(got[:, :Hkv, :bs * D], want.reshape(nb, Hkv, bs * D)), (n, Hkv, D, bs, which)
            assert not got[:, Hkv:].any() and not got[:, :, bs * D:].any()


@pytest.mark.parametrize("dtype,fp8", [("bf16", False), ("f32", False), ("bf16", True), ("f32", True)])
@pytest.mark.parametrize("layout", [B.SMART_KV_PLAIN, B.SMART_KV_INTERLEAVED])
@pytest.mark.parametrize("kind", ["prompts", "offset", "reversed", "holes"])
def test_token_runs(dtype, fp8, layout, kind):
    _check(dtype, fp8, layout, kind, ((1, 2, 64, 8), (7, 1, 8, 16), (8, 3, 64, 24), (9, 8, 128, 16), (61, 5, 128, 64), (200, 2, 72, 8)))


@pytest.mark.parametrize("dtype,fp8", [("bf16", False), ("f32", False), ("bf16", True), ("f32", True)])
@pytest.mark.parametrize("layout", [B.SMART_KV_PLAIN, B.SMART_KV_INTERLEAVED])
@pytest.mark.parametrize("kind", ["prompts", "offset", "reversed", "holes"])
def test_runs_that_move_in_chunks(dtype, fp8, layout, kind):
    """Token counts on both sides of where the chunk kernel takes over, for narrow rows (down to one chunk: most lanes have
    nothing to move) and for wide ones."""
    if layout == B.SMART_KV_PLAIN:
        sizes = ((3, 8, 128, 16), (17, 9, 128, 24), (1927, 1, 136, 24), (1928, 1, 136, 24), (32768, 1, 8, 16))
    elif fp8:
        sizes = ((12799, 1, 8, 16), (12803, 1, 8, 64))
    else:
        sizes = ((799, 4, 128, 16), (805, 4, 128, 64), (1599, 3, 24, 24), (1600, 1, 72, 8), (1606, 3, 24, 24), (1605, 1, 8, 16))
    _check(dtype, fp8, layout, kind, sizes)


def test_rows_off_the_chunks():
    """A source that is not aligned to 16 bytes, and a token stride that is no multiple of 8: the same bytes."""
    import torch
    lib = B.SmartTree(0)
    n, Hkv, D, bs, nb = 20, 2, 64, 16, 4
    src = torch.randn(n * Hkv * D + 1, device="cuda").to(torch.bfloat16)
    k, v = src[1:].view(n, Hkv, D), src[:-1].view(n, Hkv, D)
    slots = torch.arange(n, device="cuda")
    for stride in (D, D + 2):
        kc, vc = (torch.zeros((nb, Hkv, bs, stride), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        lib.kv_cache_write(k, v, slots, kc, vc, B.SMART_KV_PLAIN, bs, nb, kc.stride(0), kc.stride(1), token_stride=stride)
        for c, x in ((kc, k), (vc, v)):
            assert torch.equal(c.permute(0, 2, 1, 3).reshape(nb * bs, Hkv, stride)[:n, :, :D], x)


@pytest.mark.parametrize("dtype,fp8", [("bf16", False), ("f32", False), ("bf16", True), ("f32", True)])
@pytest.mark.parametrize("layout,pad", [(B.SMART_KV_PLAIN, 0), (B.SMART_KV_PLAIN, 2), (B.SMART_KV_INTERLEAVED, 0)])
@pytest.mark.parametrize("Hkv", [3, 8, 15])
def test_commit_of_long_paths(dtype, fp8, layout, pad, Hkv):
    """Paths of up to 128 entries (a lane per entry, three turns), refused ones among them: an entry or a block past the
    first 64 that is not there, no room in the table."""
    import torch
    lib = B.SmartTree(0)
    rng = np.random.default_rng(9)
    n, D, bs, max_depth = 128, 72, 8, 127                    # (rows of 216, 576 and 1080 elements: by element, in chunks but for fp8, in chunks)
    lens = np.array([5, 0, 9, 1, 2, 3, 200], np.int32)
    alen = np.array([127, 63, 64, 0, 100, 100, 60], np.int32)
    nseq, max_blocks = len(lens), 32
    path = np.full((nseq, max_depth + 1), -1, np.int32)
    for b in range(nseq):
        path[b, :alen[b] + 1] = np.arange(alen[b] + 1)
    path[4, 90] = n                                          # not a node
    nb = nseq * max_blocks
    table = rng.permutation(nb).reshape(nseq, max_blocks).astype(np.int32)
    table[5, (3 + 80) // bs] = nb                            # not a block
    cu = (np.arange(nseq + 1) * n).astype(np.int32)
    expect = [0, 0, 0, 0, B.SMART_ETREE, B.SMART_ETREE, B.SMART_ECAP]
    k, v = (W._normal(2, i, (nseq * n, Hkv, D), 1.0, dtype) for i in (1, 2))
    f = lambda x: (W.bf16_bits_to_f32(x) if dtype == "bf16" else x).astype(np.float32)
    val = [F.encode(f(x) / np.float32(sc)) for x, sc in ((k, 0.03), (v, 0.011))] if fp8 else [k, v]
    plain = [np.zeros((nb, Hkv, bs, D), x.dtype) for x in val]
    for b in range(nseq):
        for i in range(alen[b] + 1 if expect[b] == 0 else 0):
            pos = int(lens[b]) + i
            for p, x in zip(plain, val):
                p[table[b, pos // bs], :, pos % bs] = x[b * n + i]
    tk, tv = H.torch_elems(k, dtype, "cuda"), H.torch_elems(v, dtype, "cuda")
    shape = (nb, Hkv, bs, D + pad) if layout == B.SMART_KV_PLAIN else (nb, Hkv, bs * D)
    kc, vc = (torch.zeros(shape, dtype=torch.uint8 if fp8 else tk.dtype, device="cuda") for _ in range(2))
    t = lambda a: torch.from_numpy(a).cuda()
    scales = dict(k_scale=0.03, v_scale=0.011) if fp8 else {}
    new, status = lib.tree_commit(t(cu), t(alen), t(path), tk, tv, kc, vc, t(table), t(lens), layout, bs, nb, kc.stride(0),
                                  kc.stride(1), token_stride=D + pad, **scales)
    assert status.tolist() == expect
    assert new.tolist() == [int(x + y + 1) if e == 0 else int(x) for x, y, e in zip(lens, alen, expect)]
    for c, p, which in zip((kc, vc), plain, "kv"):
        got = c.cpu()
        got = (got if fp8 else got.view(torch.int16 if dtype == "bf16" else torch.float32)).numpy().view(p.dtype)
        if layout == B.SMART_KV_PLAIN:
            assert np.array_equal(got[..., :D], p) and not got[..., D:].any()
        else:
            assert np.array_equal(got, KL.interleave_plain_cache(p, which))
