"""Attention walks the lists it is given: a caller that leaves tiles out of a built
mask's lists gets the attention over the rest, for every pattern, dtype and entry
point, also where the library finds a pattern's tiles without the lists as long as
they are its own, and in a captured call whose lists change between replays.

Tolerances as in the attention tests: 2e-2 (bf16) and 1e-4 (f32) absolute for
outputs of N(0, 1) values, 1e-3 for lse.
"""
import copy
import types

import numpy as np
import pytest
import torch

import paper_2511_05832_amd as hla
import workloads as W
from helpers import TOL_LSE, TOL_OUT, max_abs, np64
from oracle import masks as o_masks

Pat = W.Pattern
LISTS = ("n_full", "full_idx", "n_part", "part_idx")


def test_lists_are_the_builders_until_taken():
    """Reading a list or the struct, by any name or copy, or another struct ends it;
    nothing else does. A list is an ordinary attribute after that."""
    pat = Pat("rowmajor_slide", 24, 32, 4, 4)
    for name in LISTS + ("struct",):
        mask = hla.BlockMask(pat, 128, 64, device="cpu", columns=True)
        twin = copy.copy(mask)
        assert mask.N == 0 and mask.n_qtiles == 6 and mask.totals.numel() == 2 and mask.n_full_t.numel() == 12
        assert hla._lists_of(mask).own and hla._lists_of(twin).own
        got = getattr(twin, name)
        assert not hla._lists_of(mask).own
        assert getattr(twin, name) is got and getattr(mask, name) is got
        if name != "struct":
            assert got.data_ptr() == getattr(mask.struct, name)
    mask = hla.BlockMask(pat, 128, 64, device="cpu")
    mask.struct = other = hla.BlockMaskStruct()
    assert not hla._lists_of(mask).own and hla._lists_of(mask).struct is other
    assert not hla._lists_of(hla.BlockMask(Pat("hilbert_slide", 16, 16, 9), 128, 64, device="cpu")).own
    plain = types.SimpleNamespace(struct=other)      # any object with a struct will do
    assert not hla._lists_of(plain).own and hla._lists_of(plain).struct is other


def thin(mask, rng):
    """Leave out about a third of every list's entries and all of one row's; returns
    the tiles that stay, as a boolean [n_qtiles, n_ktiles]."""
    torch.cuda.synchronize()
    kept = np.zeros((mask.n_qtiles, mask.n_ktiles), dtype=bool)
    for n_name, i_name in (("n_full", "full_idx"), ("n_part", "part_idx")):
        n, idx = getattr(mask, n_name), getattr(mask, i_name)
        nn, ii = n.cpu().numpy().copy(), idx.cpu().numpy().copy()
        for row in range(mask.n_qtiles):
            stay = [t for t in ii[row, :nn[row]] if row != 1 and rng.random() < 0.67]
            nn[row] = len(stay)
            ii[row] = -1
            ii[row, :len(stay)] = stay
            kept[row, stay] = True
        n.copy_(torch.from_numpy(nn))
        idx.copy_(torch.from_numpy(ii))
    return kept


def reference(q, k, v, scale, allowed):
    s = np.where(allowed, np64(q) @ np64(k).transpose(0, 1, 3, 2) * scale, -np.inf)
    m = np.max(s, -1, keepdims=True)
    p = np.exp(s - np.where(np.isinf(m), 0.0, m))
    l = p.sum(-1, keepdims=True)
    with np.errstate(divide="ignore"):
        lse = (np.where(np.isinf(m), 0.0, m) + np.log(l))[..., 0]
    return (p / np.where(l == 0, 1.0, l)) @ np64(v), lse


@pytest.mark.gpu
@pytest.mark.parametrize("pat", [
    Pat("rowmajor_slide", 31, 47, 8, 8), Pat("rowmajor_window", 32, 32, 8, 8),
    Pat("rowmajor_window", 33, 50, 16, 16), Pat("rowmajor_neighborhood", 24, 40, 13, 13),
    Pat("hilbert_slide", 24, 32, 100)], ids=str)
@pytest.mark.parametrize("d,tm,dtype", [(64, 128, "bf16"), (32, 64, "bf16"), (64, 64, "f32")])
def test_thinned_lists(pat, d, tm, dtype):
    B, heads, N = 1, 2, pat.N
    q, k, v = W.attn_inputs(B, heads, N, d, dtype, seed=N + d)
    scale = 1.0 / d ** 0.5
    dev = [t.cuda() for t in (q, k, v)]
    order = torch.randperm(N, generator=torch.Generator().manual_seed(N)).to(torch.int32).cuda()
    grid = [hla.scatter(t, order) for t in dev]
    mask = hla.build_block_mask(pat, tm, 64)
    dense = o_masks.dense(pat)

    def check(want, lse_want, got, lse):
        assert max_abs(np64(got), want) <= TOL_OUT[dtype] and max_abs(np64(lse), lse_want) <= TOL_LSE

    def calls():
        check(want, lse_want, *hla.attn_fwd(*dev, mask, scale))
        out, lse = hla.attn_fwd_perm(*grid, order, mask, scale)
        check(want, lse_want, out[:, :, order.long()], lse[:, :, order.long()])

    want, lse_want = reference(q, k, v, scale, dense)
    calls()
    # captured while the lists are still the builder's, replayed after they changed
    out, lse = torch.empty_like(dev[0]), torch.empty((B, heads, N), device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        hla.attn_fwd(*dev, mask, scale, out=out, lse=lse)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hla.attn_fwd(*dev, mask, scale, out=out, lse=lse)
    graph.replay()
    torch.cuda.synchronize()
    check(want, lse_want, out, lse)

    kept = thin(mask, np.random.default_rng(N + tm))
    i = np.arange(N)
    want, lse_want = reference(q, k, v, scale, dense & kept[i[:, None] // tm, i[None, :] // 64])
    calls()
    for _ in range(2):
        out.normal_()
        graph.replay()
        torch.cuda.synchronize()
        check(want, lse_want, out, lse)
