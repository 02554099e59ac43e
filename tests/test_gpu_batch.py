"""tagc_compress_ranks: the ranks' work in the same launches must leave, rank by rank, what
tagc_compress leaves -- pairs, counts and Index bit for bit -- whatever the batches are: more
ranks than one launch takes, ranks that share a workspace (they take turns), ranks with and
without a gradient accumulator side by side, on fresh and on carried pre-thresholds."""
import numpy as np
import pytest
import torch

from synth import gradients as G

pytestmark = pytest.mark.gpu


def _bucket(name, dtype, n_ranks):
    if name == "mixed":   # short and unaligned segments
        return G.small_mixed_bucket(seed=3, dtype=dtype, n_ranks=n_ranks, sizing_milli=1500)
    return G.config1(seed=5, n=(1 << 18) + 4321, n_ranks=n_ranks)    # fp32, one long segment


@pytest.mark.parametrize("name,dtype,n_ranks,layout", [
    ("mixed", G.BF16, 35, "own"), ("mixed", G.F32, 33, "pairs"), ("mixed", G.F32, 6, "acc"),
    ("long", G.F32, 5, "own"), ("long", G.F32, 7, "pairs"), ("long", G.F32, 4, "acc"),
    ("mixed", G.BF16, 1, "own"), ("long", G.F32, 3, "one")])
def test_batched_ranks_equal_ranks_one_by_one(name, dtype, n_ranks, layout):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] batch %s dtype=%d ranks=%d %s" % (name, dtype, n_ranks, layout), flush=True)
    b = _bucket(name, dtype, n_ranks)
    kw = dict(sizing_milli=b.sizing_milli, seed=9, part_unknowns=512, part_cells=1536,
              error_feedback=layout == "acc")
    ref = TagcBucket(b.segments, b.dtype, n_ranks, **kw)
    got = TagcBucket(b.segments, b.dtype, n_ranks, **kw)
    for r in range(n_ranks):
        if layout == "pairs":     # neighbours share a workspace
            got.rk[r].workspace = got.rk[r // 2 * 2].workspace
        elif layout == "one":
            got.rk[r].workspace = got.rk[0].workspace
        elif layout == "acc" and r % 3 == 1:    # no accumulator for some of the ranks
            ref.rk[r].acc = got.rk[r].acc = None
    for step in range(2):
        grads = [G.rank_gradient(b, r + 100 * step, "cuda") for r in range(n_ranks)]
        for r in range(n_ranks):
            ref.compress_index(r, grads[r])
        got.compress_index_all(grads)
        ref.aggregate_index()
        got.aggregate_index()
        for r in range(n_ranks):
            ref.compress_sketch(r)
        got.compress_sketch_all()
        torch.cuda.synchronize()
        assert got.header() == ref.header()
        for r in range(n_ranks):
            c0, c1 = ref.rank_counts(r), got.rank_counts(r)
            assert c0["total"] == c1["total"] and c0["seg"] == c1["seg"] and c1["flags"] == 0
            (i0, v0), (i1, v1) = ref.rank_pairs(r), got.rank_pairs(r)
            assert np.array_equal(i0, i1) and np.array_equal(v0.view(np.uint32), v1.view(np.uint32))
            assert np.array_equal(ref.rank_bitmap(r), got.rank_bitmap(r))
            # a cell is a float32 sum of at most a few dozen values whose order is free
            s0, s1 = ref.rank_sketch(r), got.rank_sketch(r)
            assert np.all(np.abs(s0.astype(np.float64) - s1) <= 1e-5 * np.abs(v0).max())
            if ref.rk[r].acc:
                assert np.array_equal(ref.rank_acc(r), got.rank_acc(r))
    ref.close()
    got.close()
