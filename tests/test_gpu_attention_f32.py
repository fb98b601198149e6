"""fp32 attention, forward and backward, at the edges of the 32 x 32 blocks its
kernels work in: windows and bands that cut blocks at odd positions, blocks
without any allowed pair, grid rows shorter than a block, ragged last tiles, both
head dims and query tiles, in sequence order and with the reordering fused in.

Tolerance. A score is a sum of d fp32 products: its error is at most
d * 2^-24 * sum |q k| * scale, about 2e-5 at d = 64 for N(0, 1) inputs, and moves a
weight by as much, relatively; sums over keys average such errors. The bound,
5e-5 of the largest magnitude (at least 1), is above that for outputs and
gradients alike; the plain fp32 rounding of the results is far below it.
"""
import numpy as np
import pytest
import torch

import paper_2511_05832_amd as hla
import workloads as W
from helpers import max_abs, np64
from oracle import attention as o_attn
from oracle import permute as o_perm

pytestmark = pytest.mark.gpu

REL = 5e-5
Pat = W.Pattern


@pytest.mark.parametrize("pat", [
    Pat("hilbert_window", 8, 8, 64), Pat("hilbert_window", 16, 17, 49), Pat("hilbert_slide", 32, 16, 3),
    Pat("hilbert_slide", 20, 20, 97), Pat("hilbert_neighborhood", 15, 13, 33),
    Pat("hilbert_shifted_window", 16, 32, 96, 48), Pat("rowmajor_slide", 33, 8, 2, 3),
    Pat("rowmajor_slide", 5, 96, 1, 20), Pat("rowmajor_window", 12, 40, 7, 16),
    Pat("rowmajor_neighborhood", 10, 64, 3, 33), Pat("hilbert_window", 1, 5, 2)], ids=str)
@pytest.mark.parametrize("d,tm", [(32, 64), (32, 128), (64, 64), (64, 128)])
def test_f32_blocks(pat, d, tm):
    B, heads, N = 1, 2, pat.N
    q, k, v = W.attn_inputs(B, heads, N, d, "f32", seed=N + d)
    g = torch.randn((B, heads, N, d), generator=torch.Generator().manual_seed(N))
    scale = 1.0 / d ** 0.5
    mask = hla.build_block_mask(pat, tm, 64, columns=True)
    dev = [t.cuda() for t in (q, k, v, g)]
    out, lse = hla.attn_fwd(*dev[:3], mask, scale)
    grads = hla.attn_bwd(*dev[:3], out, dev[3], lse, mask, scale)
    ref_out, ref_lse = o_attn.attention(*(np64(t) for t in (q, k, v)), pat, scale)
    ref = (ref_out, *o_attn.attention_backward(*(np64(t) for t in (q, k, v, g)), pat, scale))
    for name, got, want in zip(("out", "dq", "dk", "dv"), (out, *grads), ref):
        bound = REL * max(1.0, float(np.abs(want).max()))
        assert max_abs(np64(got), want) <= bound, (name, max_abs(np64(got), want), bound)
    assert max_abs(np64(lse), ref_lse) <= REL * max(1.0, float(np.abs(ref_lse).max()))

    # the reordering fused in gives the same bits, in the order's rows
    order = torch.randperm(N, generator=torch.Generator().manual_seed(3)).to(torch.int32)
    to_grid = [torch.from_numpy(o_perm.scatter(t.numpy(), order.numpy())).cuda() for t in (q, k, v, g)]
    order = order.cuda()
    out_p, lse_p = hla.attn_fwd_perm(*to_grid[:3], order, mask, scale)
    grads_p = hla.attn_bwd_perm(*to_grid[:3], out_p, to_grid[3], lse_p, order, mask, scale)
    for got, want in zip((out_p, lse_p, *grads_p), (out, lse, *grads)):
        assert torch.equal(got[:, :, order.long()], want)
