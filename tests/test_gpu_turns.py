"""tagc_compress_ranks with ranks that take turns (one workspace) carries pre-thresholds from rank to
rank, as one call per rank does: the same segments are re-routed, call by call."""
import numpy as np
import pytest
import torch

from synth import gradients as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("exponents", [(0, -12, 0), (0, 0, -12, -12)])
def test_turns_carry_pre_thresholds(dtype, exponents):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] turns dtype=%d %s" % (dtype, exponents), flush=True)
    n, ranks = 300_000, len(exponents)
    segs = [G.Seg(0, n, 10_000, 1, "w"), G.Seg(n, 140_000, 20_000, 1, "v")]
    td = torch.float32 if dtype == G.F32 else torch.bfloat16
    ref = TagcBucket(segs, dtype, ranks, seed=9)
    got = TagcBucket(segs, dtype, ranks, seed=9, ranks_together=1)
    gen = torch.Generator(device="cuda").manual_seed(3)
    seen = 0
    for step in range(3):
        grads = [(torch.randn(n + 140_000, generator=gen, device="cuda") * 2.0 ** e).to(td)
                 for e in exponents]
        for r in range(ranks):
            ref.compress_index(r, grads[r])
        got.compress_index_all(grads)
        torch.cuda.synchronize()
        for r in range(ranks):
            assert ref.rank_counts(r) == got.rank_counts(r)
            seen += ref.rank_counts(r)["dense_segments"]
            (i0, v0), (i1, v1) = ref.rank_pairs(r), got.rank_pairs(r)
            assert np.array_equal(i0, i1) and np.array_equal(v0, v1)
    assert seen
    ref.close()
    got.close()
