"""The candidate scan stages fewer slots at a time for plans that have other buckets in flight
(decode_workgroups) and chunks of fewer than 192 slots: runs that end with the list of chunks and runs that end
with the staging area, kept fractions on both sides of the rule, with and without an accumulator, against the
oracle and the other form's results."""
import pytest
import torch

from synth import gradients as G
from oracle import tagc_oracle as O
from paper_2504_05638_amd.bucket import TagcBucket
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


# slots per chunk of 2048 entries: 64, 160, 192 and 544
@pytest.mark.parametrize("ppm", [8_000, 33_000, 36_000, 144_000])
def test_against_oracle(ppm):
    print("\n[case] scan stage ppm=%d" % ppm, flush=True)
    n = 300_007
    b = G.Bucket("scan_stage", G.BF16, 2, [G.Seg(0, n, ppm, 1, "w")], n, 2000)
    grads = [torch.randn(n, generator=torch.Generator().manual_seed(r)).mul_(1e-3).to(torch.bfloat16)
             for r in range(2)]
    ores, tb = run_both(b, grads, seed=3, decode_workgroups=64)
    dev = [g.cuda() for g in grads]
    for _ in range(2):  # (now with a pre-threshold of its own)
        tb.run(dev)
        torch.cuda.synchronize()
        compare_all(b, ores, tb)
        assert all(tb.rank_counts(r)["dense_segments"] == 0 for r in range(2))


@pytest.mark.parametrize("ppm", [8_000, 33_000])
def test_both_forms_with_an_accumulator(ppm):
    print("\n[case] scan stage with an accumulator ppm=%d" % ppm, flush=True)
    n = 300_007
    segs = [(0, n, ppm, 1)]
    mk = lambda wgs: TagcBucket(segs, O.BF16, 1, sizing_milli=2000, error_feedback=True, decode_workgroups=wgs)
    one, two = mk(0), mk(64)
    for step in range(4):
        g = torch.randn(n, generator=torch.Generator().manual_seed(step)).mul_(1e-3).to(torch.bfloat16).cuda()
        for tb in (one, two):
            tb.compress_index(0, g)
        torch.cuda.synchronize()
        assert (one.rank_acc(0) == two.rank_acc(0)).all() and (one.rank_bitmap(0) == two.rank_bitmap(0)).all()
        for a, c in zip(one.rank_pairs(0), two.rank_pairs(0)):
            assert (a == c).all()
