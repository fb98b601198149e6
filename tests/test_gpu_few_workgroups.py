"""The bf16 forward's kernels for launches of few workgroups and for the others give
the same bits: the same slices in launches of 2, 96 and 176 heads, which lie on both
sides of every line the launcher draws (one wave per SIMD, half a wave for the
one-launch kernel, six two-wave workgroups per CU), plain, with the reordering fused in
and, on 2^k grids, as one launch; and the slices agree with the oracle (2e-2 absolute
for outputs of N(0, 1) values, 1e-3 for lse, as in the attention tests).
"""
import pytest
import torch

import paper_2511_05832_amd as hla
import workloads as W
from helpers import TOL_LSE, max_abs, np64
from oracle import attention as o_attn

pytestmark = pytest.mark.gpu

Pat = W.Pattern


@pytest.mark.parametrize("pat", [
    Pat("hilbert_window", 16, 32, 49), Pat("hilbert_window", 16, 32, 256), Pat("hilbert_slide", 16, 32, 40),
    Pat("hilbert_slide", 16, 32, 3), Pat("hilbert_neighborhood", 20, 24, 81),
    Pat("hilbert_shifted_window", 16, 31, 144, 72), Pat("hilbert_slide", 16, 16, 33),
    Pat("hilbert_window", 16, 16, 80), Pat("hilbert_shifted_window", 16, 16, 48, 17)], ids=str)
@pytest.mark.parametrize("d,tm", [(32, 64), (32, 128), (64, 64), (64, 128)])
def test_same_bits_at_every_launch_size(pat, d, tm):
    N, most = pat.N, 176
    q, k, v = W.attn_inputs(1, most, N, d, "bf16", seed=N + d + tm)
    scale = 1.0 / d ** 0.5
    mask = hla.build_block_mask(pat, tm, 64)
    order = hla.hilbert_perm(pat.H, pat.W)[0]
    dev = [t.cuda() for t in (q, k, v)]
    grid = [hla.scatter(t, order) for t in dev]
    one_launch = pat.H == pat.W
    ref_out, ref_lse = o_attn.attention(*(np64(t[:, :2]) for t in (q, k, v)), pat, scale)
    first = None
    for heads in (2, 96, most):
        out, lse = hla.attn_fwd(*(t[:, :heads].contiguous() for t in dev), mask, scale)
        part = [t[:, :heads].contiguous() for t in grid]
        got = [hla.attn_fwd_perm(*part, order, mask, scale)]
        if one_launch:
            got.append(hla.attn_fwd_hilbert(*part, pat, tm, 64, scale))
        for out_p, lse_p in got:
            assert torch.equal(hla.gather(out_p, order), out) and torch.equal(lse_p[:, :, order.long()], lse), heads
        if first is None:
            first = out, lse
            assert max_abs(np64(out), ref_out) <= 2e-2 and max_abs(np64(lse), ref_lse) <= TOL_LSE
        assert torch.equal(out[:, :2], first[0]) and torch.equal(lse[:, :2], first[1]), heads
