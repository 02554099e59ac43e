"""Buckets with segments on both of the sparsifier's routes, on both sides of the line between the
forms of the ordered output they take (most pairs from the dense route, or not: tiles staged in LDS
or stored entry by entry), with few candidates per chunk and with hundreds; first as planned, then
with the candidate-route segment re-routed, its scale having fallen.  Pairs and Index bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from synth import gradients as G
from tests.helpers import oracle_config, oracle_segments

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("fast_ppm", [10_000, 100_000])
@pytest.mark.parametrize("dense", ["few", "half", "most"])
def test_both_routes(dtype, fast_ppm, dense):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] both routes dtype=%d fast=%d dense=%s" % (dtype, fast_ppm, dense), flush=True)
    n_fast, ranks = 300_000, 2
    k_fast = n_fast * fast_ppm // 1_000_000
    n_dense = 2 * k_fast                            # ("half": as many pairs as the other segment)
    ppm = {"few": 20_000, "half": 500_000, "most": 600_000}[dense]
    segs = [G.Seg(0, n_fast, fast_ppm, 1, "fast"),
            G.Seg(n_fast + 1, n_dense, ppm, 1, "dense"),
            G.Seg(n_fast + n_dense + 3, 9_001, 0, 1, "nothing kept"),
            G.Seg(n_fast + n_dense + 9_007, 1_003, 1_000_000, 1, "all kept")]
    total = segs[-1].offset + segs[-1].length
    b = G.Bucket("both", dtype, ranks, segs, total, 1500)
    rng = np.random.default_rng(31)
    td = torch.float32 if dtype == G.F32 else torch.bfloat16
    tb = TagcBucket(b.segments, b.dtype, ranks, sizing_milli=1500, seed=3)
    for scale in (1.0, 2.0 ** -12):
        grads = [torch.from_numpy(rng.standard_normal(total).astype(np.float32) *
                                  np.float32(scale)).to(td) for _ in range(ranks)]
        tb.compress_index_all([g.cuda() for g in grads])
        torch.cuda.synchronize()
        for r in range(ranks):
            want = O.sparsify(G.to_numpy_raw(grads[r]), oracle_config(b), oracle_segments(b))
            cnt = tb.rank_counts(r)
            assert cnt["flags"] == 0 and cnt["seg"] == list(want.seg_cnt)
            assert cnt["dense_segments"] == (2 if scale == 1.0 else 3)
            idx, val = tb.rank_pairs(r)
            assert np.array_equal(idx, want.idx)
            assert np.array_equal(val.view(np.uint32), want.val.view(np.uint32))
            assert np.array_equal(tb.rank_bitmap(r), want.bitmap[:tb.sizes.bitmap_words])
    tb.close()
