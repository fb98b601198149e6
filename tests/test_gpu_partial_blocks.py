"""Partial tiles in 32-key and 32-row blocks: windows, bands and neighbourhoods whose
edges leave a wave none, one or both blocks of a tile, forward (plain, reordering
fused, position bias) and backward, both head dims and query tiles, against the
oracle. Tolerances as in the attention and backward tests: 2e-2 absolute for
outputs, 2e-2 of the largest magnitude (at least 1) for gradients, 1e-3 for lse.
"""
import numpy as np
import pytest
import torch

import paper_2511_05832_amd as hla
import workloads as W
from helpers import TOL_LSE, max_abs, np64
from oracle import attention as o_attn

pytestmark = pytest.mark.gpu

Pat = W.Pattern


@pytest.mark.parametrize("pat", [
    Pat("hilbert_window", 16, 32, 32), Pat("hilbert_window", 16, 32, 96), Pat("hilbert_window", 20, 20, 33),
    Pat("hilbert_slide", 16, 32, 31), Pat("hilbert_slide", 16, 32, 32), Pat("hilbert_slide", 16, 32, 95),
    Pat("hilbert_neighborhood", 16, 32, 65), Pat("hilbert_shifted_window", 16, 32, 160, 31),
    Pat("rowmajor_slide", 8, 64, 1, 15)], ids=str)
@pytest.mark.parametrize("d,tm", [(32, 64), (64, 128), (64, 64), (32, 128)])
def test_partial_blocks(pat, d, tm):
    B, heads, N = 1, 2, pat.N
    q, k, v = W.attn_inputs(B, heads, N, d, "bf16", seed=N + d + tm)
    gen = torch.Generator().manual_seed(N)
    g = torch.randn((B, heads, N, d), generator=gen).to(torch.bfloat16)
    rpb = torch.randn((heads, 2 * pat.H - 1, 2 * pat.W - 1), generator=gen)
    scale = 1.0 / d ** 0.5
    mask = hla.build_block_mask(pat, tm, 64, columns=True)
    dev = [t.cuda() for t in (q, k, v, g)]
    qn, kn, vn, gn = (np64(t) for t in (q, k, v, g))
    out, lse = hla.attn_fwd(*dev[:3], mask, scale)
    ref_out, ref_lse = o_attn.attention(qn, kn, vn, pat, scale)
    assert max_abs(np64(out), ref_out) <= 2e-2 and max_abs(np64(lse), ref_lse) <= TOL_LSE
    grads = hla.attn_bwd(*dev[:3], out, dev[3], lse, mask, scale)
    for got, want in zip(grads, o_attn.attention_backward(qn, kn, vn, gn, pat, scale)):
        assert max_abs(np64(got), want) <= 2e-2 * max(1.0, float(np.abs(want).max()))
    # the reordering fused in: the same bits in the order's rows
    order = torch.randperm(N, generator=gen).to(torch.int32).cuda()
    grid = [hla.scatter(t, order) for t in dev]
    out_p, lse_p = hla.attn_fwd_perm(*grid[:3], order, mask, scale)
    grads_p = hla.attn_bwd_perm(*grid[:3], out_p, grid[3], lse_p, order, mask, scale)
    for got, want in zip((out_p, lse_p, *grads_p), (out, lse, *grads)):
        assert torch.equal(got[:, :, order.long()], want)
    # position bias (the order: the identity grid)
    ids = torch.arange(N, dtype=torch.int32).cuda()
    out_b, lse_b = hla.attn_fwd_rpb(*dev[:3], ids, rpb.cuda(), mask, scale)
    ref_out, ref_lse = o_attn.attention(qn, kn, vn, pat, scale, rpb=(np64(rpb), np.arange(N)))
    assert max_abs(np64(out_b), ref_out) <= 2e-2 and max_abs(np64(lse_b), ref_lse) <= TOL_LSE
