"""Row-major patterns walked over patches of the grid: grids whose sides are below,
at and past a patch, rectangles that end inside, at and past patch edges, radii
and kernels from none to the whole grid, windows that straddle patches, both head
dims and query tiles, in sequence order and with the reordering fused in. The
results are compared with the oracle and with the walk over the tile lists (the
position-bias entry point takes it; its table is zero here).

Tolerance: 2e-2 absolute for the outputs (bf16 weights and results of N(0, 1)
values) and 1e-3 for lse, as in the attention tests; the two walks sum the same
weights in another order, so they agree to one bf16 rounding of the output and of
the weights (2^-8 each, of values up to 4) and to fp32 sums in lse.
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
CASES = [
    Pat("rowmajor_slide", 24, 32, 0, 0), Pat("rowmajor_slide", 24, 32, 1, 2), Pat("rowmajor_slide", 25, 33, 4, 4),
    Pat("rowmajor_slide", 31, 47, 8, 8), Pat("rowmajor_slide", 40, 24, 7, 9), Pat("rowmajor_slide", 33, 16, 30, 3),
    Pat("rowmajor_slide", 17, 40, 40, 40), Pat("rowmajor_window", 32, 32, 8, 8), Pat("rowmajor_window", 30, 45, 7, 7),
    Pat("rowmajor_window", 33, 50, 16, 16), Pat("rowmajor_window", 20, 64, 3, 21),
    Pat("rowmajor_neighborhood", 24, 40, 7, 7), Pat("rowmajor_neighborhood", 19, 29, 13, 5),
    Pat("rowmajor_neighborhood", 26, 26, 26, 26), Pat("rowmajor_neighborhood", 48, 10, 9, 10),
    Pat("rowmajor_slide", 64, 7, 3, 2), Pat("rowmajor_window", 96, 5, 4, 4), Pat("rowmajor_slide", 1, 200, 0, 5)]


@pytest.mark.parametrize("pat", CASES, ids=str)
@pytest.mark.parametrize("d,tm", [(64, 128), (64, 64), (32, 128), (32, 64)])
def test_patches(pat, d, tm):
    B, heads, N = 1, 2, pat.N
    q, k, v = W.attn_inputs(B, heads, N, d, "bf16", seed=N + d)
    scale = 1.0 / d ** 0.5
    mask = hla.build_block_mask(pat, tm, 64)
    dev = [t.cuda() for t in (q, k, v)]
    out, lse = hla.attn_fwd(*dev, mask, scale)
    ref_out, ref_lse = o_attn.attention(*(np64(t) for t in (q, k, v)), pat, scale)
    assert max_abs(np64(out), ref_out) <= 2e-2 and max_abs(np64(lse), ref_lse) <= TOL_LSE
    zero = torch.zeros((heads, 2 * pat.H - 1, 2 * pat.W - 1), device="cuda")
    out_l, lse_l = hla.attn_fwd_rpb(*dev, None, zero, mask, scale)
    assert max_abs(np64(out), np64(out_l)) <= 2e-2 and max_abs(np64(lse), np64(lse_l)) <= 1e-5
    order = torch.randperm(N, generator=torch.Generator().manual_seed(N)).to(torch.int32).cuda()
    out_p, lse_p = hla.attn_fwd_perm(*(hla.scatter(t, order) for t in dev), order, mask, scale)
    assert torch.equal(out_p[:, :, order.long()], out) and torch.equal(lse_p[:, :, order.long()], lse)
