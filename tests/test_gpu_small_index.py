"""Indexes of up to 4096 words that the layout merges itself: sizes around a vector, a group of 64 words, a chunk of 1024
and the limit, in the three ways of merging, against the oracle; one word more takes a merge of its own, which the
profile shows."""
import numpy as np
import pytest
import torch

from paper_2504_05638_amd import binding as B
from synth import gradients as G
from oracle import tagc_oracle as O
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [1, 3, 5, 64, 65, 1023, 1025, 2048, 4095, 4096, 4097])
@pytest.mark.parametrize("ranks,mode", [(1, O.INDEX_OR1), (3, O.INDEX_OR1), (5, O.INDEX_ADD1), (2, O.INDEX_ADD4), (9, O.INDEX_OR1),
                                        (8, O.INDEX_ADD4), (9, O.INDEX_ADD4)])
def test_merged_by_the_layout(words, ranks, mode):
    print("\n[case] small index words=%d ranks=%d mode=%d" % (words, ranks, mode), flush=True)
    n = 32 * words - 5  # (padding bits at the end)
    b = G.Bucket("small_index", G.F32, ranks, [G.Seg(0, n, 60_000, 1, "a")], n, 1500)
    rng = np.random.default_rng(words)
    grads = [torch.from_numpy(rng.integers(-200, 201, n).astype(np.float32)) for _ in range(ranks)]
    ores, tb = run_both(b, grads, seed=4, index_mode=mode)
    compare_all(b, ores, tb, exact_values=True)
    B.tagc_profile_enable(True)
    try:
        tb.run([g.cuda() for g in grads])
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    bytes_ = ranks * words * (16 if mode == O.INDEX_ADD4 else 4)
    assert ("index_or" in B.tagc_profile_read()) == (words > 4096 or bytes_ > 128 * 1024 or
                                                            (mode == O.INDEX_ADD4 and ranks > 8))
    compare_all(b, ores, tb, exact_values=True)
    tb.close()


# The merged Index in the place of a rank's own: merged by a launch of its own, whatever the size
@pytest.mark.parametrize("words", [1, 65, 4096])
@pytest.mark.parametrize("rank", [0, 2])
@pytest.mark.parametrize("mode", [O.INDEX_OR1, O.INDEX_ADD1])
def test_merged_in_place(words, rank, mode):
    print("\n[case] small index in place words=%d rank=%d mode=%d" % (words, rank, mode), flush=True)
    n, ranks = 32 * words - 5, 3
    b = G.Bucket("small_index", G.F32, ranks, [G.Seg(0, n, 60_000, 1, "a")], n, 1500)
    rng = np.random.default_rng(words)
    grads = [torch.from_numpy(rng.integers(-200, 201, n).astype(np.float32)) for _ in range(ranks)]
    ores, tb = run_both(b, grads, seed=4, index_mode=mode)
    tb.shared.bitmap = tb.rk[rank].bitmap
    B.tagc_profile_enable(True)
    try:
        tb.run([g.cuda() for g in grads])
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    assert "index_or" in B.tagc_profile_read()
    assert np.array_equal(tb.rank_bitmap(rank), ores.bitmap[:words])
    tb.sh_bitmap.copy_(tb._rk_tensors[rank]["bitmap"][:tb.sh_bitmap.numel()])
    local = ores.ranks[rank].bitmap[:words].copy()
    tb._rk_tensors[rank]["bitmap"][:4 * words].copy_(torch.from_numpy(local.view(np.uint8)))
    compare_all(b, ores, tb, exact_values=True)
    tb.close()
