"""fp32: the threshold's low 16 key bits counted from the gradient itself: long segments off every
16-byte boundary (several vectors per thread, a ragged end), and long ones that were re-routed
because their scale fell since the pre-threshold was tuned, alone and beside each other, over more
ranks than one; ties in thousands.  Pairs and Index bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from synth import gradients as G
from tests.helpers import oracle_config, oracle_segments

pytestmark = pytest.mark.gpu

_SEGS = {"planned": [(1, 3_000_003, 400_000)],
         "rerouted": [(0, 2_000_000, 10_000)],
         "both": [(0, 700_000, 10_000), (700_001, 1_100_001, 400_000), (1_800_004, 300_000, 20_000)]}


@pytest.mark.parametrize("name", list(_SEGS))
@pytest.mark.parametrize("ties", [False, True])
def test_low_key_bits_of_the_dense_route(name, ties):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] refine dense %s ties=%d" % (name, ties), flush=True)
    segs = [G.Seg(o, n, k, 1, "s%d" % i) for i, (o, n, k) in enumerate(_SEGS[name])]
    total, ranks = segs[-1].offset + segs[-1].length, 3
    b = G.Bucket(name, G.F32, ranks, segs, total, 1500)
    rng = np.random.default_rng(21)
    tb = TagcBucket(b.segments, b.dtype, ranks, sizing_milli=1500, seed=3)
    for scale in (1.0, 2.0 ** -12):
        grads = []
        for r in range(ranks):
            g = rng.standard_normal(total).astype(np.float32)
            grads.append(torch.from_numpy((np.round(g * 64) / 64 if ties else g) * np.float32(scale)))
        tb.compress_index_all([g.cuda() for g in grads])
        torch.cuda.synchronize()
        for r in range(ranks):
            want = O.sparsify(G.to_numpy_raw(grads[r]), oracle_config(b), oracle_segments(b))
            cnt = tb.rank_counts(r)
            assert cnt["flags"] == 0 and cnt["seg"] == list(want.seg_cnt)
            assert cnt["dense_segments"] == (len(segs) if scale < 1 else name != "rerouted")
            idx, val = tb.rank_pairs(r)
            assert np.array_equal(idx, want.idx)
            assert np.array_equal(val.view(np.uint32), want.val.view(np.uint32))
            assert np.array_equal(tb.rank_bitmap(r), want.bitmap[:tb.sizes.bitmap_words])
    tb.close()
