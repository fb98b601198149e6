"""The tiled projection kernel at the edges of its tiles: token counts below, at
and past a tile of 64 and 128 tokens, every feature-tile width (F a multiple of
192, of 128, of 64 only), the smallest and largest K, both head dims, enough
tokens for 128-token tiles and too few, with and without an order.

Tolerance: one bf16 rounding of the result (2^-9 relative) plus fp32 sums of K
products (K * 2^-24 relative to the sum of magnitudes, below 2^-14 here): 2^-8 of
the largest magnitude bounds both.
"""
import pytest
import torch

import paper_2511_05832_amd as hla

pytestmark = pytest.mark.gpu


def close(got, ref):
    err = float((got.double() - ref).abs().max())
    assert err <= 2 ** -8 * float(ref.abs().max()) + 1e-6, err


@pytest.mark.parametrize("heads,d,B,N,c_out", [
    (2, 32, 1, 1, 64), (2, 32, 1, 63, 64), (1, 64, 1, 64, 128), (4, 32, 1, 65, 320), (2, 64, 3, 43, 192),
    (8, 64, 1, 127, 448), (16, 32, 1, 128, 512), (10, 32, 1, 129, 640), (7, 64, 2, 500, 384),
    (8, 64, 2, 4099, 512), (12, 32, 7, 1201, 384), (2, 32, 5, 8191, 64), (4, 64, 3, 9000, 128)], ids=str)
@pytest.mark.parametrize("ordered", [False, True])
def test_projection_tiles(heads, d, B, N, c_out, ordered):
    C = heads * d
    g = torch.Generator(device="cuda").manual_seed(heads * N + c_out)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)

    x, wq, wp, o = normal(B, N, C), normal(3 * C, C, std=0.05), normal(c_out, C, std=0.05), normal(B, heads, N, d)
    order = torch.randperm(N, generator=g, device="cuda").to(torch.int32) if ordered else None
    rows = order.long() if ordered else torch.arange(N, device="cuda")
    ref = (x[:, rows].double() @ wq.double().T).reshape(B, N, 3, heads, d).permute(2, 0, 3, 1, 4)
    for got, want in zip(hla.qkv_proj(x, wq, heads, order=order), ref):
        close(got, want)
    ref = o.double().permute(0, 2, 1, 3).reshape(B, N, C) @ wp.double().T
    y = hla.out_proj(o, wp, order=order)
    close(y[:, rows], ref)
