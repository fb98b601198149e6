"""The bench's FLOP counts: allowed pairs of every row-major pattern against the
oracle's dense mask, the listed tiles for the kernels that walk the lists, and each
rate published under the name of what it is counted over."""
import types

import pytest

import bench
import workloads as W
from oracle import masks as o_masks

Pat = W.Pattern


@pytest.mark.parametrize("pat", [
    Pat("rowmajor_window", 13, 10, 4, 3), Pat("rowmajor_window", 8, 16, 8, 20), Pat("rowmajor_slide", 9, 14, 2, 5),
    Pat("rowmajor_slide", 6, 5, 0, 9), Pat("rowmajor_neighborhood", 11, 9, 5, 4),
    Pat("rowmajor_neighborhood", 7, 7, 7, 1)], ids=str)
def test_rowmajor_pairs(pat):
    assert bench.rowmajor_pairs(pat) == int(o_masks.dense(pat).sum())


def test_rowmajor_pairs_refuses_other_patterns():
    with pytest.raises(ValueError):
        bench.rowmajor_pairs(Pat("hilbert_slide", 8, 8, 3))


@pytest.mark.parametrize("w", [W.C3, W.C3_ROWMAJOR], ids=lambda w: w.name)
def test_flops_and_their_names(w):
    pipe = object.__new__(bench.AttnPipeline)
    pipe.w, pipe.hilbert = w, w.pattern.hilbert
    pipe.mask = types.SimpleNamespace(host_totals=lambda: (3, 4))
    pipe.timer = types.SimpleNamespace(pairs={}, mean_ms=lambda name: 1.0)
    tiles = 4.0 * w.tile_m * w.tile_n * w.d * 7 * w.B * w.heads
    assert pipe.tile_flops() == (tiles, 3, 4)
    res = bench.summarize(pipe, (1.0, 1.0, {"graph": 1.0, "stream": 1.0}))
    assert res["tile_flops"] == tiles
    if w.pattern.hilbert:
        assert res["attn_tflops_nonempty_tiles"] == pytest.approx(tiles / 1e9) and "attn_tflops_allowed_pairs" not in res
    else:
        pairs = 4.0 * w.d * bench.rowmajor_pairs(w.pattern) * w.B * w.heads
        assert res["attn_tflops_allowed_pairs"] == pytest.approx(pairs / 1e9) and "attn_tflops_nonempty_tiles" not in res
