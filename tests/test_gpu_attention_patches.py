"""Row-major patterns walked over patches of the grid: grids whose sides are below,
at and past a patch, rectangles that end inside, at and past patch edges, radii
and kernels from none to the whole grid, windows that straddle patches, both head
dims and query tiles, in sequence order and with the reordering fused in. Every case
runs over patches and over the tile lists, each named in the call, and both are
compared with the oracle and with each other.

Tolerance: 2e-2 absolute for the outputs (bf16 weights and results of N(0, 1)
values) and 1e-3 for lse, as in the attention tests; the two walks sum the same
weights in another order, so they agree to one bf16 rounding of the output and of
the weights (2^-8 each, of values up to 4) and to fp32 sums in lse.
"""
import ctypes

import pytest
import torch

import paper_2511_05832_amd as hla
import workloads as W
from helpers import TOL_LSE, max_abs, np64
from oracle import attention as o_attn

pytestmark = pytest.mark.gpu

Pat = W.Pattern
CASES = [
    Pat("rowmajor_slide", 24, 32, 0, 0), Pat("rowmajor_slide", 24, 32, 1, 2), Pat("rowmajor_slide", 25, 33, 4, 4),
    Pat("rowmajor_slide", 31, 47, 8, 8), Pat("rowmajor_slide", 40, 24, 7, 9), Pat("rowmajor_slide", 33, 16, 30, 3),
    Pat("rowmajor_slide", 17, 40, 40, 40), Pat("rowmajor_window", 32, 32, 8, 8), Pat("rowmajor_window", 30, 45, 7, 7),
    Pat("rowmajor_window", 33, 50, 16, 16), Pat("rowmajor_window", 20, 64, 3, 21),
    Pat("rowmajor_neighborhood", 24, 40, 7, 7), Pat("rowmajor_neighborhood", 19, 29, 13, 5),
    Pat("rowmajor_neighborhood", 26, 26, 26, 26), Pat("rowmajor_neighborhood", 48, 10, 9, 10),
    Pat("rowmajor_slide", 64, 7, 3, 2), Pat("rowmajor_window", 96, 5, 4, 4), Pat("rowmajor_slide", 1, 200, 0, 5)]


def forward(walk, q, k, v, order, mask, scale):
    """hla_attn_fwd_pattern with a walk of its own choice (the call fails where the
    pattern cannot walk patches, so a result by patches is one)."""
    B, heads, N, d = q.shape
    out, lse = torch.empty_like(q), torch.empty((B, heads, N), device="cuda")
    hla._check(hla.lib().hla_attn_fwd_pattern(
        hla._ptr(q), hla._ptr(k), hla._ptr(v), hla._ptr(order), ctypes.byref(mask.struct), hla._ptr(out),
        hla._ptr(lse), B, heads, N, d, hla.HLA_BF16, scale, walk, hla._stream(q)))
    return out, lse


@pytest.mark.parametrize("pat", CASES, ids=str)
@pytest.mark.parametrize("d,tm", [(64, 128), (64, 64), (32, 128), (32, 64)])
def test_patches(pat, d, tm):
    B, heads, N = 1, 2, pat.N
    q, k, v = W.attn_inputs(B, heads, N, d, "bf16", seed=N + d)
    scale = 1.0 / d ** 0.5
    mask = hla.build_block_mask(pat, tm, 64)
    dev = [t.cuda() for t in (q, k, v)]
    order = torch.randperm(N, generator=torch.Generator().manual_seed(N)).to(torch.int32).cuda()
    grid = [hla.scatter(t, order) for t in dev]
    rows = order.long()
    auto, auto_lse = hla.attn_fwd(*dev, mask, scale)       # before the struct is taken
    auto_p, auto_lse_p = hla.attn_fwd_perm(*grid, order, mask, scale)
    out, lse = forward(hla.HLA_WALK_PATCHES, *dev, None, mask, scale)
    out_l, lse_l = forward(hla.HLA_WALK_LISTS, *dev, None, mask, scale)
    ref_out, ref_lse = o_attn.attention(*(np64(t) for t in (q, k, v)), pat, scale)
    for o, l in ((out, lse), (out_l, lse_l)):
        assert max_abs(np64(o), ref_out) <= 2e-2 and max_abs(np64(l), ref_lse) <= TOL_LSE
    assert max_abs(np64(out), np64(out_l)) <= 2e-2 and max_abs(np64(lse), np64(lse_l)) <= 1e-5
    # the reordering fused in: the same bits in the order's rows
    for walk, want, want_lse in ((hla.HLA_WALK_PATCHES, out, lse), (hla.HLA_WALK_LISTS, out_l, lse_l)):
        out_p, lse_p = forward(walk, *grid, order, mask, scale)
        assert torch.equal(out_p[:, :, rows], want) and torch.equal(lse_p[:, :, rows], want_lse)
    # left to the library: one of the two, the same one with and without an order
    assert any(torch.equal(auto, o) and torch.equal(auto_lse, l) for o, l in ((out, lse), (out_l, lse_l)))
    assert torch.equal(auto_p[:, :, rows], auto) and torch.equal(auto_lse_p[:, :, rows], auto_lse)
    # and a mask whose lists a caller has taken walks the lists
    again, again_lse = hla.attn_fwd(*dev, mask, scale)
    assert torch.equal(again, out_l) and torch.equal(again_lse, lse_l)


@pytest.mark.parametrize("pat,tm,patches", [
    (Pat("rowmajor_slide", 48, 56, 12, 12), 64, True), (Pat("rowmajor_window", 32, 64, 8, 8), 128, True),
    (Pat("rowmajor_neighborhood", 71, 33, 13, 13), 64, True),
    # fewer tiles by patches, but the fullest patch has 9 against 7
    (Pat("rowmajor_neighborhood", 32, 32, 13, 13), 64, False),
    (Pat("rowmajor_slide", 64, 64, 3, 3), 64, False)], ids=str)
def test_the_choice_of_walk(pat, tm, patches):
    """Which walk a call takes, the same for 2 slices and for 96 of them."""
    N, d = pat.N, 32
    q, k, v = (t.cuda() for t in W.attn_inputs(1, 96, N, d, "bf16", seed=N))
    mask = hla.build_block_mask(pat, tm, 64)
    auto = [hla.attn_fwd(*(t[:, :heads].contiguous() for t in (q, k, v)), mask)[0] for heads in (2, 96)]
    walks = [forward(walk, q, k, v, None, mask, d ** -0.5)[0] for walk in (hla.HLA_WALK_LISTS, hla.HLA_WALK_PATCHES)]
    assert not torch.equal(*walks)
    assert torch.equal(auto[1], walks[patches]) and torch.equal(auto[0], auto[1][:, :2])
