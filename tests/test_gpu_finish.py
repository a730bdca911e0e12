"""The one-launch form of the interleaved kernels (bf16, head dim 128, block size 16; bf16 and fp8 caches), which evaluates
the tree part on the matrix cores and merges a segment's pieces where the last of them ends, and the two-launch form, taken
where few sequences have room for long prefixes: both against the general kernel, which holds probabilities in binary32.

Tolerance, element by element, as for one and two row tiles of the fp8 cache (test_gpu_fp8_row_tiles): every probability,
those of the tree's own keys included, is rounded to bf16 (u = 2^-8), which moves an output by at most u times the weighted
mean of |V|, and both sides round the output once."""
import numpy as np
import pytest

from paper_2604_09731_amd import binding as B
from tests.test_gpu_tiled_attention import Inputs

pytestmark = pytest.mark.gpu

WIDE = 1000          # spare columns of the block table: room for 16000 tokens
#        tree sizes (edges of the classes and of the 32-key tiles), prefixes (edges of the 32-key tiles, none), heads
SHAPES = [([1, 8, 9, 16, 17, 64, 65, 128], [0, 1, 31, 32, 33, 517, 1000, 95], 8, 2),
          ([1, 31, 32, 33, 64, 65, 128], [500, 0, 64, 700, 2, 33, 0], 2, 2),
          ([4, 5, 9, 10, 36, 37, 74], [900, 33, 95, 0, 700, 1, 300], 14, 2)]


def bound_of(x, lib, ref):
    v, v_tree = x.v, x.v_tree
    x.v, x.v_tree = (v & 0x7F) if x.kw else v.abs(), v_tree.abs()
    spread = x.run(lib, general=True)[0].double()
    x.v, x.v_tree = v, v_tree
    u = 2.0 ** -8
    return (u * (1 + u) + 2.0 ** -16) * spread + 2 * u * (1 + u) * ref.double().abs()


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("workers", [0, 1, 3, 40, 300])
def test_both_forms_equal_the_general_kernel(shape, workers, fp8):
    """Segments of one worker, of two and of up to 30; shares that end in a prefix, between it and its tree part, and
    inside a tile; the plan made by the workgroups (few sequences) and by a kernel of its own (more than 64)."""
    import torch
    sizes, lens, Hq, Hkv = SHAPES[shape]
    lib = B.SmartTree(0)
    for times, spare in ((1, 1), (1, WIDE), (10, 1)):
        x = Inputs(sizes * times, lens * times, Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=shape + workers,
                   spare_columns=spare)
        ref, ref_lse = x.run(lib, general=True)
        bound = bound_of(x, lib, ref)
        lib.set_option(B.SMART_OPT_TVA_WORKERS, workers)
        for static in (False, True):
            status = torch.full((len(sizes) * times,), -3, dtype=torch.int32, device="cuda")
            out, lse = x.run(lib, static=static, status=status)
            assert bool(((out.double() - ref.double()).abs() <= bound).all())      # (false for NaN)
            assert float((lse - ref_lse).abs().max()) <= 1e-3
            assert not status.any()
            for _ in range(3):           # pieces are merged in a fixed order, whoever comes last: the same bits every time
                again, again_lse = x.run(lib, static=static)
                assert torch.equal(again, out) and torch.equal(again_lse, lse)
        lib.set_option(B.SMART_OPT_TVA_WORKERS, 0)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("lens,size,Hq,Hkv", [([64, 0, 0, 0], 4, 16, 4), ([40] + [0] * 6, 3, 28, 4), ([128, 32] + [0] * 6, 8, 8, 2),
                                              ([33] + [0] * 14, 100, 2, 2), ([0] * 9 + [64] + [0] * 5, 50, 2, 2)])
def test_mostly_empty_prefixes_under_a_wide_table(lens, size, Hq, Hkv, fp8):
    """Two launches, and more segments than units of prefix: no partial is merged that this call did not write.  A larger call
    leaves its own in the workspace first; values of its cache are far from those of the calls behind it."""
    lib = B.SmartTree(0)
    x = Inputs([size] * len(lens), lens, Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=len(lens), spare_columns=WIDE)
    big = Inputs([size] * len(lens), [3000] * len(lens), Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, False, seed=1,
                 spare_columns=WIDE)
    big.v.mul_(1e4)
    ref, ref_lse = x.run(lib, general=True)
    bound = bound_of(x, lib, ref)
    for static in (False, True):
        big.run(lib, static=static)
        out, lse = x.run(lib, static=static)
        assert bool(((out.double() - ref.double()).abs() <= bound).all())
        assert float((lse - ref_lse).abs().max()) <= 1e-3


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("size,Hq,Hkv", [(8, 8, 2), (16, 8, 2), (50, 4, 4), (64, 8, 2), (128, 8, 2)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_what_one_node_holds_reaches_only_its_descendants(bad, size, Hq, Hkv, fp8):
    """A value, and the key, of one node: rows that do not see it keep their bits; rows that do are what the general kernel
    makes of them (row groups of every class, both tiles of tree keys and the four of the largest tree)."""
    import torch
    lib = B.SmartTree(0)
    x = Inputs([size, 3], [200, 40], Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=size)
    _, _, _, mask, _ = lib.tree_pack(x.cu, x.parent, x.len)
    words = mask.cpu().numpy().view(np.uint64).reshape(-1, 2)
    clean, _ = x.run(lib)
    for node in (size // 3, size - 1):
        sees = torch.from_numpy((words[:size, node // 64] >> np.uint64(node % 64)) & np.uint64(1) == 1).cuda()
        v = x.v_tree.clone()
        x.v_tree[node, :, 5], x.v_tree[node, :, 77] = bad, -bad
        out, _ = x.run(lib)
        ref, _ = x.run(lib, general=True)
        assert torch.equal(out[:size][~sees], clean[:size][~sees]) and torch.equal(out[size:], clean[size:])
        got, want = out[:size][sees], ref[:size][sees]
        assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(got[torch.isinf(got)], want[torch.isinf(want)])
        others = [d for d in range(128) if d not in (5, 77)]
        assert torch.equal(got[..., others], clean[:size][sees][..., others])
        x.v_tree = v
        k = x.k_tree.clone()
        x.k_tree[node, :, 9] = bad
        out, _ = x.run(lib)
        assert torch.equal(out[:size][~sees], clean[:size][~sees]) and torch.equal(out[size:], clean[size:])
        x.k_tree = k


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("size,prefix", [(33, 20), (50, 0), (50, 20), (64, 100), (100, 20)])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_bad_values_in_several_tiles_of_tree_keys(bad, size, prefix, fp8):
    """One in each tile of 32 tree keys, and prefixes so short that the wavefronts that carry those tiles have no other key:
    each row is what the general kernel makes of it."""
    import torch
    lib = B.SmartTree(0)
    x = Inputs([size, 3], [prefix, 40], 4, 4, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=size)
    for at, node in enumerate(range(5, size, 27)):
        x.v_tree[node, :, 7 * at + 1], x.v_tree[node, :, 7 * at + 2] = bad, -bad
    out, _ = x.run(lib)
    ref, _ = x.run(lib, general=True)
    assert torch.isnan(ref).any() if np.isnan(bad) else torch.isinf(ref).any()
    assert torch.equal(torch.isnan(out), torch.isnan(ref)) and torch.equal(out[torch.isinf(out)], ref[torch.isinf(ref)])


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("size,Hq,Hkv", [(16, 8, 2), (50, 4, 4), (64, 8, 2), (128, 8, 2)])
def test_an_infinite_value_of_the_key_with_all_the_weight(size, Hq, Hkv, fp8):
    """A node whose score is 181 above all others it sees (their probabilities are zero in binary32) and whose value is
    infinite: its row is infinite there, not NaN."""
    import torch
    lib = B.SmartTree(0)
    x = Inputs([size, 3], [200, 40], Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=size)
    x.k_tree.mul_(0.01)
    for node in (size // 2 + 15 if size > 32 else size // 2, size - 1):
        q, k, v = x.q.clone(), x.k_tree.clone(), x.v_tree.clone()
        x.q[node], x.k_tree[node], x.v_tree[node, :, 5] = 8.0, 2.0, np.inf
        out, _ = x.run(lib)
        assert bool((out[node, :, 5] == np.inf).all())
        assert torch.isfinite(out[node][:, [d for d in range(128) if d != 5]]).all()
        x.q, x.k_tree, x.v_tree = q, k, v


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("size,Hq,Hkv", [(1, 32, 8), (7, 32, 8), (10, 32, 8), (40, 8, 2), (64, 8, 2), (128, 8, 2)])
def test_the_largest_probability_of_a_tree_tile_is_not_rounded(size, Hq, Hkv, fp8):
    """One prefix key of score and value 0 and tree values of 1: a root's row, which sees one tree key, is p / (1 + p).  Nothing
    is rounded to 16 bits but the output (half a unit in its last place)."""
    lib = B.SmartTree(0)
    x = Inputs([size] * 40, [1] * 40, Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, fp8, seed=size)
    x.k.zero_()
    x.v.zero_()
    x.v_tree.fill_(1)
    s = (x.q[::size].double().view(40, Hkv, -1, 128) * x.k_tree[::size, :, None].double()).sum(-1) / np.sqrt(128)
    p = s.exp().view(40, Hq, 1)
    ref = p / (1 + p)
    out, lse = x.run(lib)
    bound = 2.0 ** (ref.log2().floor() - 8) + 1e-5 * ref           # (1e-5: scores and exponentials in binary32)
    assert bool(((out[::size].double() - ref).abs() <= bound).all())
    assert float((lse[::size].double() - (1 + p[..., 0]).log()).abs().max()) <= 1e-5


@pytest.mark.parametrize("scale", [1e-39, 2e-38, 1e-30])
@pytest.mark.parametrize("size,Hq,Hkv", [(7, 32, 8), (40, 8, 2), (128, 8, 2)])
def test_a_softmax_scale_near_zero(size, Hq, Hkv, scale):
    """Every key a row sees has the same weight, also where the scale's reciprocal is no binary32: the two sides differ by a
    unit of bf16 at most, and by what sums in another order move in binary32."""
    lib = B.SmartTree(0)
    x = Inputs([size] * 40, [40] * 40, Hq, Hkv, 128, 16, "bf16", B.SMART_KV_INTERLEAVED, seed=size)
    _, _, _, mask, _ = lib.tree_pack(x.cu, x.parent, x.len)
    got = {}
    for general in (1, 0):
        lib.set_option(B.SMART_OPT_TVA_FORCE_GENERAL, general)
        got[general] = lib.tree_verify_attention(x.q, x.k_tree, x.v_tree, x.k, x.v, x.table, x.len, x.cu, mask, scale, x.layout,
                                                 block_size=16, want_lse=True)
    (out, lse), (ref, ref_lse) = got[0], got[1]
    assert bool(((out.double() - ref.double()).abs() <= 2.0 ** -7 * ref.double().abs() + 1e-5).all())
    assert float((lse - ref_lse).abs().max()) <= 1e-5
